"""Calls at the ends of what the entry points accept: shared buffers, values
that are not finite, the largest grids, very small steps, and calls that a
stream capture interrupts."""
import ctypes as C
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


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("at", [0, 3 * 96 * 80 * 56 // 4 - 512 * 384])
def test_projection_over_its_own_volume(noalloc, at):
    """The projection written over the start or the middle of the volume: the
    same as into a buffer of its own (the FP32 projection parity bound)."""
    L = _lib()
    g = S.Grid((96, 80, 56), (3.0, 3.0, 4.0))
    G = S.Geom(0.4, 512, 384, 0.9, 0.9, 1.5)
    x = torch.zeros(max(g.N, at + 512 * 384), device=DEV)
    vol = x[:g.N].view(g.shape)
    vol.copy_(torch.tensor(S.seeded(3, g.shape, "uniform"), dtype=torch.float32))
    want = L.forward_project(g, G, vol.clone()).cpu().numpy()
    out = x[at:at + 512 * 384].view(384, 512)
    (L.forward_project_noalloc if noalloc else L.forward_project)(g, G, vol, out)
    assert rel_l2(out.cpu().numpy(), want) <= 1e-5


@pytest.mark.parametrize("value", [math.inf, -math.inf, math.nan])
@pytest.mark.parametrize("step", [1.0, 3.5])
@pytest.mark.parametrize("n,du", [((37, 34, 19), 3.1), ((130, 90, 61), 9.0)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_backprojection_of_a_pixel_that_is_not_finite(value, step, n, du, dtype):
    """A residual that is infinite or NaN reaches the voxels its ray's samples
    weigh, and no other: the rest are those of the residual with that pixel at
    zero, within the backprojection parity bounds.  (Weights below 1e-5 are left out of the check: in FP32
    a weight of zero may come out as a rounding error and the other way round.)"""
    L = _lib()
    g = S.Grid(n, (2.0, 2.0, 2.0))
    G = S.Geom(math.radians(25.0), 37, 29, du, du, step, off_u=0.3, off_v=-0.2)
    r = torch.tensor(S.seeded(6, (29, 37)), dtype=dtype)
    for iv, iu in ((14, 18), (5, 9)):
        one = np.zeros((29, 37))
        one[iv, iu] = 1.0
        weight = oracle.backproject(g, G, one)
        r[iv, iu] = 0.0
        rest = L.backproject_residual(g, G, r.to(DEV)).cpu().numpy()
        r[iv, iu] = value
        got = L.backproject_residual(g, G, r.to(DEV)).cpu().numpy()
        assert (weight > 1e-5).sum() > 20
        reached = got[weight > 1e-5]
        assert np.isnan(reached).all() if math.isnan(value) else (reached == value).all()
        assert rel_l2(got[weight == 0], rest[weight == 0]) <= (1e-5 if dtype == torch.float32 else 1e-12)
        r[iv, iu] = 0.0
