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


@pytest.mark.parametrize("compute", [torch.float32, torch.float64])
def test_infinite_gradient_of_an_infinite_voxel(compute):
    """A reference image of -inf at its last corner, moved by less than a voxel
    against every axis: the derivatives there are -inf, so with rising fields,
    a bright measurement and a, b > 0 every term of J and of its gradient is
    +inf, and none is NaN."""
    L = _lib()
    g = S.Grid((12, 10, 8), (2.0, 2.5, 3.0))
    f = torch.zeros(g.shape, dtype=compute)
    f[-1, -1, -1] = -math.inf
    mean = torch.full((3,) + g.shape, -0.7, dtype=compute)
    U = torch.full((1, 3) + g.shape, 0.1, dtype=compute)
    G = S.Geom(0.3, 40, 33, 1.7, 1.7, 0.9, off_u=0.21, off_v=0.13)
    ctx = L.Context(g, L.DeviceModel(mean.to(DEV), U.to(DEV)), f.to(DEV), compute=compute)
    y = torch.ones((33, 40), dtype=compute, device=DEV)
    J, grad = ctx.cost_grad(y, G, [0.5], 0.9, 0.1)
    ctx.close()
    assert J == math.inf and grad[0] == math.inf


@pytest.mark.parametrize("ang", [20.0, 110.0, 200.0])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_backprojection_of_millions_of_samples(ang, dtype):
    """A step so small that a ray takes over a million samples on either side
    of a brick's middle.  A voxel sums up to 400 000 of them in a chain, each
    addition within half an ulp of the sum: 400 000 x 2^-24 or 2^-53, and 1e-11
    for the positions (1e-16 x 1e6 samples x 0.1) in FP64."""
    L = _lib()
    g = S.Grid((5, 4, 3), (2.0, 2.0, 2.0))
    G = S.Geom(math.radians(ang), 3, 2, 4.0, 4.0, 1.2e-5, sad=100.0, sdd=150.0, off_u=0.3)
    r_t, r = rounded(S.seeded(9, (2, 3)), dtype)
    bp = L.backproject_residual(g, G, r_t.to(DEV)).cpu().numpy()
    bound = 4e5 * 2.0 ** -24 if dtype == torch.float32 else 4e5 * 2.0 ** -53 + 1e-11
    assert rel_l2(bp, oracle.backproject(g, G, r)) <= bound


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("nz", [65533, 65535])
def test_projection_of_the_longest_grid(nz, noalloc):
    """As many slices as a grid may have, in FP64, which marches a padded copy:
    the projection parity bound."""
    L = _lib()
    g = S.Grid((3, 2, nz), (2.0, 2.0, 0.01))
    G = S.Geom(0.5, 24, 30, 0.4, 25.0, 0.7)
    x = S.seeded(5, g.shape, "uniform")
    out = torch.empty((30, 24), dtype=torch.float64, device=DEV)
    vol = torch.tensor(x, dtype=torch.float64, device=DEV)
    (L.forward_project_noalloc if noalloc else L.forward_project)(g, G, vol, out)
    assert rel_l2(out.cpu().numpy(), oracle.project(g, G, x)) <= 1e-12


def _hip():
    """The HIP runtime that this process has loaded."""
    for line in open("/proc/self/maps"):
        if "libamdhip64" in line:
            return C.CDLL(line.split()[-1])
    raise RuntimeError("no HIP runtime loaded")


@pytest.mark.parametrize("mode", ["fused", "adjoint"])
def test_evaluation_after_one_that_a_capture_refused(mode):
    """An evaluation waits for its sums, so on a capturing stream it fails, and
    what it enqueued there never runs.  The next one on the same context must
    not count on it: its result is a fresh context's."""
    L = _lib()
    hip = _hip()
    grad_mode = L.GRAD_FUSED if mode == "fused" else L.GRAD_ADJOINT
    g = S.Grid((24, 20, 16), (3.0, 3.0, 3.0))
    G = S.Geom(math.radians(35.0), 33, 40, 2.7, 2.0, 1.5)
    f = torch.tensor(S.phantom(g, seed=8), dtype=torch.float32, device=DEV)
    z = np.indices(g.shape) / 7.0
    mean = torch.tensor(np.stack([2.0 * np.sin(z[a] + a) for a in range(3)]), dtype=torch.float32, device=DEV)
    U = torch.tensor(np.stack([np.sin(z[a] * 1.3) for a in range(3)])[None], dtype=torch.float32, device=DEV)
    y = torch.ones((40, 33), device=DEV)
    model = L.DeviceModel(mean, U)
    ctx = L.Context(g, model, f)
    want = ctx.cost_grad(y, G, [0.4], 0.9, 0.01, mode=grad_mode)
    ctx.close()
    # freed device memory that does not hold zeros
    sizes = [256] * 64 + [1 << 15] * 8 + [1 << 17] * 8
    p = [C.c_void_p() for _ in sizes]
    for q, n in zip(p, sizes):
        assert hip.hipMalloc(C.byref(q), C.c_size_t(n)) == 0
        assert hip.hipMemset(q, 0xA5, C.c_size_t(n)) == 0
    torch.cuda.synchronize()
    for q in p:
        assert hip.hipFree(q) == 0
    ctx = L.Context(g, model, f)
    small = S.Geom(0.5, 33, 40, 2.7, 2.0, 1e-6)
    with pytest.raises(L.PCRError):   # refused, once the image's support is known
        ctx.cost_grad(y, small, [0.4], 0.9, 0.01, mode=grad_mode)
    s = torch.cuda.Stream()
    assert hip.hipStreamBeginCapture(C.c_void_p(s.cuda_stream), 2) == 0   # relaxed
    with pytest.raises(L.PCRError):
        ctx.cost_grad(y, G, [0.4], 0.9, 0.01, mode=grad_mode, stream=s)
    graph = C.c_void_p()
    hip.hipStreamEndCapture(C.c_void_p(s.cuda_stream), C.byref(graph))   # (invalid by now)
    hip.hipGetLastError()
    for _ in range(3):
        got = ctx.cost_grad(y, G, [0.4], 0.9, 0.01, mode=grad_mode)
        assert got[0] == want[0] and np.array_equal(got[1], want[1])
    ctx.close()


# Captured projections, in a process of their own (the library keeps what the
# first calls of a process and of a thread set up).
_CAPTURED = """
import torch
from paper_1004_0014_amd import _lib as L, synth as S
g = S.Grid((40, 36, 28), (2.0, 2.0, 2.0))
fine, coarse = S.Geom(0.4, 72, 52, 1.5, 1.5, 1.0), S.Geom(0.4, 9, 7, 30.0, 30.0, 1.0)
x = torch.tensor(S.phantom(g, seed=2), dtype=torch.%s, device="cuda")
xf, pf = x.float(), torch.empty((52, 72), device="cuda")
G = %s
p = torch.full((G.nv, G.nu), float("nan"), dtype=x.dtype, device="cuda")
%s
s = torch.cuda.Stream()
s.wait_stream(torch.cuda.current_stream())
graph = torch.cuda.CUDAGraph()
with torch.cuda.graph(graph, stream=s):
    %s(g, G, x, p, stream=s)
want = L.forward_project(g, G, x)
assert want.abs().max() > 0
%s
for k in range(3):
    p.fill_(float("nan"))
    graph.replay()
    torch.cuda.synchronize()
    assert torch.equal(p, want), k
print("replays equal")
"""


def _captured(dtype, geom, before, call, after=""):
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", _CAPTURED % (dtype, geom, before, call, after)], cwd=root, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "replays equal" in r.stdout, r.stdout + r.stderr


def test_first_padded_noalloc_projection_under_capture():
    """A process whose first allocation-free projection needs no padded copy
    and whose second, which does, is captured."""
    _captured("float64", "fine", "L.forward_project_noalloc(g, fine, xf, pf)", "L.forward_project_noalloc")


def test_graph_keeps_the_scratch_that_a_later_call_outgrows():
    """A captured projection, then one of a larger grid, which needs a larger
    copy: the graph's replays still have theirs."""
    _captured("float64", "fine", "L.forward_project(g, G, x)", "L.forward_project", """
big = S.Grid((60, 50, 40), (2.0, 2.0, 2.0))
y = torch.tensor(S.phantom(big, seed=3), dtype=torch.float64, device="cuda")
q = L.forward_project(big, G, y)
junk = [torch.full((40 * 36 * 28,), 7.0, dtype=torch.float64, device="cuda") for _ in range(64)]
""")


@pytest.mark.parametrize("before", ["", "L.forward_project(S.Grid((8, 8, 8), (2.0, 2.0, 2.0)), coarse, x[:8, :8, :8].contiguous())"])
def test_padded_projection_captured_after_one_that_is_not(before):
    """A projection that needs no padded copy, then, captured, one of the same
    grid that does, in a thread with no scratch or a smaller one: its room is
    there, as a capture cannot allocate it."""
    _captured("float32", "coarse", before + "\nL.forward_project(g, fine, x, pf)", "L.forward_project")


@pytest.mark.parametrize("n,nu,nv,du", [
    ((40, 33, 21), 5, 4, 30.0),       # few bricks under few rays: 4 x 4 columns
    ((40, 33, 21), 40, 33, 4.0),      # near the rule's line, on one side in FP32
    ((40, 33, 21), 90, 70, 1.7),      # and on the other
    ((10, 102, 110), 13, 1, 9.0),     # no ray for most bricks
])
@pytest.mark.parametrize("ang", [20.0, 110.0])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_backprojection_by_the_rays_of_a_column(n, nu, nv, du, ang, dtype):
    """Few bricks with few and many rays, which decide the brick's shape: the
    backprojection parity bounds."""
    L = _lib()
    g = S.Grid(n, (2.0, 2.0, 2.5))
    G = S.Geom(math.radians(ang), nu, nv, du, du, 1.0, off_u=0.3)
    r_t, r = rounded(S.seeded(4, (nv, nu)), dtype)
    bp = L.backproject_residual(g, G, r_t.to(DEV)).cpu().numpy()
    assert rel_l2(bp, oracle.backproject(g, G, r)) <= (1e-5 if dtype == torch.float32 else 1e-12)


@pytest.mark.parametrize("K", [1, 2, 3, 4, 5, 6, 8])
@pytest.mark.parametrize("storage", [torch.float32, torch.bfloat16])
def test_localisation_by_field_count(K, storage):
    """Localisation with every count of fields an instance takes: FP64 on both
    sides, so the points agree within the fixed point's tolerance of 1e-9 mm."""
    L = _lib()
    g = S.Grid((14, 11, 9), (2.0, 2.5, 3.0))
    z = np.indices(g.shape) / 9.0
    mean_t, mean = rounded(np.stack([2.0 * np.sin(z[a] + a) for a in range(3)]), storage)
    U_t, U = rounded(np.stack([np.stack([np.cos(z[(a + k) % 3] * (1 + 0.2 * k) + a) for a in range(3)]) for k in range(K)]), storage)
    w = 0.6 * np.random.default_rng(K).uniform(-1.0, 1.0, K) / K
    p = (3.1, -2.2, 1.7)
    got, st, it = L.localize_tumor(g, L.DeviceModel(mean_t.to(DEV), U_t.to(DEV)), list(w), p, tol=1e-9)
    want = oracle.localize(g, mean, U, w, p, tol=1e-9)[0]
    assert st == L.PCR_OK and it > 2
    np.testing.assert_allclose(got, want, rtol=0, atol=2e-9)


@pytest.mark.parametrize("ang", [0.3, 1.9])
def test_f64_samples_do_not_move_with_the_detector(ang):
    """The rays of a small detector, which sixteen threads share, and the same
    rays within a large one, which four do, take their samples at the same
    points: with the source a kilometre away, where a position's rounding
    shows, the projections differ by the order of up to 60 additions at most
    (60 x 2^-53 < 1e-14)."""
    L = _lib()
    g = S.Grid((21, 18, 15), (1.0, 1.0, 1.0))
    small = S.Geom(ang, 8, 6, 2.0, 2.0, 0.75, sad=1.0e6, sdd=1.5e6)
    large = S.Geom(ang, 144, 128, 2.0, 2.0, 0.75, sad=1.0e6, sdd=1.5e6)
    x = torch.tensor(S.seeded(2, g.shape, "uniform"), dtype=torch.float64, device=DEV)
    p = L.forward_project(g, small, x).cpu().numpy()
    q = L.forward_project(g, large, x).cpu().numpy()[61:67, 68:76]
    assert np.abs(q).max() > 0
    assert rel_l2(p, q) <= 1e-14


@pytest.mark.parametrize("shift", [0.0, 0.49, -0.51, -1.0, 1.0])
@pytest.mark.parametrize("n", [(1, 1, 1), (67, 3, 2), (130, 6, 5)])
def test_warp_at_and_beyond_the_faces(n, shift):
    """Voxels displaced to the image's faces, just inside, just outside and far
    beyond, mixed within a wave: values and tangents (through the gradient's
    contraction) are the oracle's, 1e-5 of the image and of the gradient, whose
    terms add up without cancelling (rising image and fields)."""
    L = _lib()
    g = S.Grid(n, (2.0, 2.0, 2.0))
    z = np.indices(g.shape)[::-1]
    f_t, f = rounded(1.0 + z[0] + 2.0 * z[1] + 3.0 * z[2], torch.float32)
    rng = np.random.default_rng(3)
    far = rng.choice([0.0, 1.0, 40.0], size=(3,) + g.shape, p=[0.4, 0.4, 0.2]) * np.array(n)[:, None, None, None]
    x_t, x = rounded(2.0 * (far * rng.choice([-1.0, 1.0], size=far.shape) + shift + 0.001), torch.float32)
    got = L.warp_volume(g, f_t.to(DEV), x_t.to(DEV)).cpu().numpy()
    assert np.linalg.norm(got - oracle.warp(g, f, x)) <= 1e-5 * np.linalg.norm(f)
    U_t, U = rounded(np.full((1, 3) + g.shape, 0.5), torch.float32)
    gv = torch.ones(g.shape, device=DEV)
    model = L.DeviceModel(x_t.to(DEV), U_t.to(DEV))
    grad = L.warp_contract(g, model, f_t.to(DEV), [0.0], gv)[0]
    jac = oracle.warp_jacobian(g, f, x)
    assert abs(grad - (jac * U[0]).sum()) <= 1e-5 * np.abs(jac * U[0]).sum()
