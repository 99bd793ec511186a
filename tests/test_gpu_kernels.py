"""Edges of the kernels' tilings and dispatch rules, against the FP64 oracle."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_1004_0014_amd import synth as S
from helpers import rel_l2, rounded

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _lib():
    from paper_1004_0014_amd import _lib as L
    return L


@pytest.mark.parametrize("n,sp,nu,nv,du,step,ang", [
    ((300, 9, 7), (0.12, 6.0, 6.0), 24, 18, 2.4, 3.0, 0.0),     # box rows of more than 64 cells
    ((9, 300, 7), (6.0, 0.12, 6.0), 24, 18, 2.4, 3.0, 90.0),    # the same along the other axis
    ((70, 66, 3), (1.0, 1.0, 30.0), 33, 17, 1.5, 0.5, 41.0),    # flat boxes: few rows
    ((5, 4, 90), (20.0, 20.0, 1.0), 19, 65, 1.5, 0.5, 200.0),   # boxes of short rows, many slices
    ((40, 40, 40), (2.0, 2.0, 2.0), 8, 6, 40.0, 1.0, 30.0),     # no box fits: the L1 gather
    ((40, 40, 40), (2.0, 2.0, 2.0), 67, 50, 2.0, 1.0, 30.0),    # ragged detector tiles
])
def test_staged_march_box_shapes(n, sp, nu, nv, du, step, ang):
    """The staged march's boxes of cells in all their shapes; FP32 sums of a
    few hundred samples: the projection parity bound of 1e-5."""
    L = _lib()
    g = S.Grid(n, sp)
    G = S.Geom(math.radians(ang), nu, nv, du, du, step, off_u=0.3, off_v=-0.4)
    x_t, x = rounded(S.seeded(3, g.shape, "uniform"), torch.float32)
    p = L.forward_project(g, G, x_t.to(DEV)).cpu().numpy()
    assert rel_l2(p, oracle.project(g, G, x)) <= 1e-5
