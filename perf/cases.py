"""The work this library is used for, as timed cases.

A case is one pass through public entry points on a seeded thorax-like
phantom, a seeded smooth motion model and a cone-beam geometry.  `op` says
which entry points:

  solve      Context.reconstruct: one frame's solve from the previous frame's
             w, with the tumour localised
  cost_grad  Context.cost_grad: J and its gradient, what each line-search trial
             and any outside optimiser evaluates (mode 0 fused, 1 paper order)
  project    forward_project of a volume
  autograd   autograd.project forward and backward (gradients in w and f0)
  volume     dvf_compose + warp_volume: the reconstructed image of a solved w
  pca        pca_train: the motion model from the training deformations
  serve      Server: several patients' frames through the batching engine

Sizes are those of the tiny, differentiation, paper-scale and precision
configurations, of the serving mix (up to 512 x 512 x 160 voxels, K = 5,
1024 x 768 pixels), or odd ones between them.
"""
from __future__ import annotations

import math
import random

import torch

from paper_1004_0014_amd import _lib, autograd
from paper_1004_0014_amd.synth import Geom, Grid

_DT = {"f32": torch.float32, "f64": torch.float64, "bf16": torch.bfloat16, "f16": torch.float16}
_SIZE = {"f32": 4, "f64": 8, "bf16": 2, "f16": 2}
_SAD, _SDD = 1000.0, 1500.0
_A, _B = 1.1, 0.05              # intensity fit of the measured projection
_AMPS = (10.0, 3.0, 1.5, 1.0, 0.8)   # mm per mode, as of breathing motion


def _case(name, op, n, fov, det, width, angle, K=3, storage="f32", compute="f32", **more):
    c = dict(op=op, nx=n[0], ny=n[1], nz=n[2], fov_xy=fov[0], fov_z=fov[1], nu=det[0], nv=det[1],
             width=width, angle=angle, K=K, storage=storage, compute=compute)
    c.update(more)
    return dict(name=name, **c) if name else c


def listed():
    paper = ((256, 256, 100), (480.0, 250.0), (512, 384), 397.3)
    precision = ((256, 256, 128), (480.0, 320.0), (512, 384), 397.3)
    return [
        # the smallest call: a coarse volume, latency and launches count
        _case("solve_tiny", "solve", (64, 64, 64), (256.0, 256.0), (128, 96), 204.8, 30.0),
        # one frame of the paper's setting
        _case("solve_paper", "solve", *paper, 57.0),
        # gradient of a mid-size volume with five modes, near the y axis
        _case("grad_mid_k5", "cost_grad", (128, 128, 128), (384.0, 384.0), (256, 192), 397.3, 95.0, K=5),
        # 16-bit model storage at the precision configuration
        _case("grad_bf16_k4", "cost_grad", *precision, 200.0, K=4, storage="bf16"),
        # the serving mix's largest stream
        _case("grad_largest", "cost_grad", (512, 512, 160), (480.0, 320.0), (1024, 768), 397.0, 20.0,
              K=5, storage="bf16"),
        # the gradient in the paper's order (backprojection, contraction)
        _case("grad_paper_order", "cost_grad", *paper, 120.0, mode=1),
        # a digitally reconstructed radiograph of a volume
        _case("project_paper", "project", *paper, 330.0),
        # FP64 on an odd grid and detector, as gradient checks run it
        _case("project_f64_odd", "project", (101, 93, 77), (300.0, 231.0), (203, 151), 300.0, 250.0,
              compute="f64"),
        # training through the projector: forward and both gradients
        _case("autograd_paper", "autograd", *paper, 15.0),
        # the reconstructed volume of a frame, odd sizes, FP16 model
        _case("volume_f16_odd", "volume", (255, 251, 99), (480.0, 250.0), (1, 1), 1.0, 0.0,
              storage="f16"),
        # motion model from nine registered phases
        _case("pca_paper", "pca", (256, 256, 100), (480.0, 250.0), (1, 1), 1.0, 0.0, J=9),
        # six patients, two frames each, through four slots
        _case("serve_mix", "serve", (256, 256, 128), (480.0, 320.0), (512, 384), 397.0, 40.0, K=4,
              storage="bf16", streams=6, frames=2),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["solve", "solve", "cost_grad", "cost_grad", "cost_grad", "project", "project",
                     "autograd", "volume", "pca"])
    xy = _log(rng, 48, 400 if op == "cost_grad" else 256)
    n = (xy, max(32, xy + rng.randint(-9, 9)), _log(rng, 32, 140))
    fov = (rng.uniform(250.0, 480.0), rng.uniform(200.0, 320.0))
    nu = _log(rng, 96, 900 if op == "cost_grad" else 512)
    det = (nu, max(48, int(0.75 * nu) + rng.randint(-7, 7)))
    K = rng.randint(1, 5)
    storage = rng.choice(["f32", "f32", "bf16", "f16"]) if op in ("cost_grad", "volume") else "f32"
    more, compute = {}, "f32"
    if op == "cost_grad" and rng.random() < 0.25:
        more["mode"] = 1
    if op == "project" and rng.random() < 0.3:
        compute = "f64"
    if op == "pca":
        more["J"] = rng.randint(6, 12)
        K = min(K, 4)
    return _case("", op, n, fov, det, rng.uniform(230.0, 400.0), rng.uniform(0.0, 360.0), K, storage,
                 compute, **more)


# ------------------------------------------------------------ inputs -------
def _grid(c):
    return Grid((c["nx"], c["ny"], c["nz"]),
                (c["fov_xy"] / c["nx"], c["fov_xy"] / c["ny"], c["fov_z"] / c["nz"]))


def _geom(c, turn=0.0):
    d = c["width"] / c["nu"]
    return Geom(math.radians(c["angle"] + turn), c["nu"], c["nv"], d, d, 0.5 * min(_grid(c).spacing),
                _SAD, _SDD)


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _mesh(g):
    ax = [g.origin[a] + g.spacing[a] * torch.arange(g.n[a], device="cuda", dtype=torch.float32)
          for a in range(3)]
    return ax[0][None, None, :], ax[1][None, :, None], ax[2][:, None, None]


def _phantom(g, seed):
    """Body and lungs as ellipsoids (1/mm), a 10 mm tumour, smooth texture."""
    L, (x, y, z), gen = g.fov, _mesh(g), _gen(seed)
    j = (0.05 * torch.rand(3, generator=gen, device="cuda")).tolist()
    mu = torch.zeros(g.shape, device="cuda")

    def paint(c, s, v):
        q = ((x - c[0]) / s[0]) ** 2 + ((y - c[1]) / s[1]) ** 2 + ((z - c[2]) / s[2]) ** 2
        mu.masked_fill_(q <= 1.0, v)

    paint((0, 0, 0), ((0.38 + j[0]) * L[0], (0.28 + j[1]) * L[1], 0.60 * L[2]), 0.02)
    for side in (1, -1):
        paint((side * 0.17 * L[0], 0.02 * L[1], 0.05 * L[2]),
              (0.13 * L[0], (0.18 + j[2]) * L[1], 0.30 * L[2]), 0.004)
    paint(_tumour(g), (10.0, 10.0, 10.0), 0.02)
    t = torch.randn(g.shape, generator=gen, device="cuda")
    t = torch.nn.functional.avg_pool3d(t[None, None], 3, 1, 1, count_include_pad=True)[0, 0]
    return (mu * (1.0 + 0.05 * t / t.std())).contiguous()


def _tumour(g):
    return (-0.17 * g.fov[0], 0.02 * g.fov[1], -0.05 * g.fov[2])


def _patterns(g, K, seed):
    """K smooth motion fields [K][3][nz][ny][nx] (mm), strongest first, decaying
    laterally; SI and AP motion dominate."""
    x, y, z = _mesh(g)
    gen = _gen(seed + 77)
    env = torch.exp(-(x / (0.35 * g.fov[0])) ** 2)
    P = torch.empty((K, 3) + g.shape, device="cuda")
    for k in range(K):
        for a, s in enumerate((0.12, 0.35, 1.0)):
            f = torch.randn(6, generator=gen, device="cuda").tolist()
            s = s if a == 2 or k % 2 == 0 else 1.35 - s
            ph = (1.0 + 0.6 * k) * (f[0] * x / g.fov[0] + f[1] * y / g.fov[1] + (1.0 + f[2]) * z / g.fov[2])
            P[k, a] = _AMPS[k] * s * env * (torch.sin(2.0 * ph + f[3]) if k else 1.0 + 0.2 * torch.sin(ph))
    return P


def _model(c, seed):
    """mean [3][N], orthonormal U [K][3][N] (FP32) and the K x K factor that
    maps pattern amplitudes to w."""
    g, K = _grid(c), c["K"]
    P = _patterns(g, K, seed).view(K, -1)
    Q = torch.empty((K, K), dtype=torch.float64, device="cuda")
    for i in range(K):
        for j in range(i + 1):
            Q[i, j] = Q[j, i] = sum((a.double() * b.double()).sum()
                                    for a, b in zip(P[i].split(1 << 24), P[j].split(1 << 24)))
    Lc = torch.linalg.cholesky(Q.cpu())
    Z = torch.linalg.inv(Lc)                       # U = Z P
    U = torch.stack([sum(float(Z[k, j]) * P[j] for j in range(k + 1)) for k in range(K)])
    mean = sum(0.4 * (-0.5) ** j * P[j] for j in range(K))
    return mean.view((3,) + g.shape), U.view((K, 3) + g.shape), Lc.T


def _w(c, seed, Lt):
    """A frame's w and the previous frame's (the warm start)."""
    r = random.Random(int(seed) * 7 + 1)
    now = [r.uniform(0.5, 1.0) * (-1) ** k for k in range(c["K"])]
    before = [v - 0.25 * r.uniform(0.5, 1.0) for v in now]
    f = lambda v: (Lt @ torch.tensor(v, dtype=torch.float64)).tolist()  # noqa: E731
    return f(now), f(before)


def _interp(vol, q):
    """Trilinear interpolation of vol [nz][ny][nx] at index points q [..., 3]
    (x, y, z), zero outside (differentiable in both)."""
    n = torch.tensor(vol.shape[::-1], device=q.device, dtype=q.dtype)
    s = (2.0 * q / (n - 1) - 1.0).reshape(1, 1, 1, -1, 3)
    v = torch.nn.functional.grid_sample(vol[None, None], s, mode="bilinear", padding_mode="zeros",
                                        align_corners=True)
    return v.reshape(q.shape[:-1])


def _points(g, dvf):
    """Index points voxel + displacement [nz][ny][nx][3]."""
    i = [torch.arange(g.n[a], device="cuda", dtype=dvf.dtype) for a in range(3)]
    base = (i[0][None, None, :], i[1][None, :, None], i[2][:, None, None])
    return torch.stack([base[a] + dvf[a] / g.spacing[a] for a in range(3)], dim=-1)


def _compose(mean, U, w):
    return mean + sum(w[k] * U[k] for k in range(U.shape[0]))


def _rays(g, G, dtype, rows):
    """Index points of the samples of detector rows `rows`, [rows][nu][n][3]:
    every ray's t = n step from the source, n over a range that covers the
    grid."""
    d = dict(device="cuda", dtype=dtype)
    st, ct = math.sin(G.angle), math.cos(G.angle)
    src = torch.tensor([G.sad * st, -G.sad * ct, 0.0], **d)
    ctr = torch.tensor([-(G.sdd - G.sad) * st, (G.sdd - G.sad) * ct, 0.0], **d)
    u = (torch.arange(G.nu, **d) - 0.5 * (G.nu - 1)) * G.du
    v = (torch.tensor([float(r) for r in rows], **d) - 0.5 * (G.nv - 1)) * G.dv
    D = (ctr - src) + u[None, :, None] * torch.tensor([ct, st, 0.0], **d) \
        + v[:, None, None] * torch.tensor([0.0, 0.0, 1.0], **d)
    D = D / D.norm(dim=-1, keepdim=True)
    R = 0.5 * math.sqrt(sum((f + 2 * s) ** 2 for f, s in zip(g.fov, g.spacing)))
    n = torch.arange(int((G.sad - R) / G.step), int((G.sad + R) / G.step) + 2, **d)
    p = src + (n * G.step)[:, None] * D[:, :, None, :]
    return (p - torch.tensor(g.origin, **d)) / torch.tensor(g.spacing, **d)


def _row_blocks(g, G):
    per = G.nu * 2 * math.sqrt(sum(f * f for f in g.fov)) / G.step
    k = max(1, int(2.0e7 / per))
    return [range(r, min(G.nv, r + k)) for r in range(0, G.nv, k)]


def _project(g, G, vol):
    return torch.cat([G.step * _interp(vol, _rays(g, G, vol.dtype, r)).sum(-1) for r in _row_blocks(g, G)])


def _backproject(g, G, resid):
    vol = torch.zeros(g.shape, device="cuda", dtype=resid.dtype, requires_grad=True)
    out = torch.zeros_like(vol)
    for r in _row_blocks(g, G):
        p = G.step * _interp(vol, _rays(g, G, resid.dtype, r)).sum(-1)
        out += torch.autograd.grad(p, vol, resid[r.start:r.stop])[0]
    return out


def _measured(g, G, f0, mean, U, w, seed):
    """A measured projection of the moved phantom, 0.2 % noise."""
    p = _project(g, G, _interp(f0, _points(g, _compose(mean, U, w))))
    noise = torch.randn(p.shape, generator=_gen(seed + 5), device="cuda")
    return ((p - _B) / _A + 0.002 * float(p.max()) * noise).contiguous()


def _stored(c, t):
    """A field stack in the case's storage type, FP16 divided by its maxima."""
    if c["storage"] != "f16":
        return t.to(_DT[c["storage"]]).contiguous(), None
    s = [max(float(u.abs().max()), 1e-30) for u in t]
    return torch.stack([u / v for u, v in zip(t, s)]).half().contiguous(), s


def _streams(c):
    """The serving mix: each stream's own sizes, up to the case's."""
    r = random.Random(c["nx"] + 31 * c["streams"])
    out = []
    for i in range(c["streams"]):
        f = 1.0 if i == 0 else r.uniform(0.4, 1.0)
        xy, nu = int(c["nx"] * f) // 16 * 16, int(c["nu"] * r.uniform(0.5, 1.0)) // 32 * 32
        out.append(dict(c, op="solve", nx=xy, ny=xy, nz=int(c["nz"] * f) // 8 * 8, nu=nu, nv=nu * 3 // 4,
                        K=r.randint(2, c["K"]), angle=c["angle"] + 50.0 * i))
    return out


def _opts(c, w, w0):
    # a frame's budget of eight iterations, about what a warm start takes
    step = 0.5 * math.sqrt(sum((a - b) ** 2 for a, b in zip(w, w0))) or 1.0
    return _lib.default_opts(max_iter=8, step0=step, localize=1, p_ref_mm=_tumour(_grid(c)))


def _parts(c, seed, frames=1):
    """What an evaluation needs: phantom, model as stored, w, measurement (and
    later frames', each a degree and a step of the motion on)."""
    g, G = _grid(c), _geom(c)
    f0 = _phantom(g, seed)
    mean, U, Lt = _model(c, seed)
    w, w0 = _w(c, seed, Lt)
    shown = [(_geom(c, float(i)), [b + 0.7 * i * (b - a) for a, b in zip(w0, w)]) for i in range(frames)]
    ys = [(_measured(g, Gi, f0, mean, U, wi, seed + 13 * i), Gi) for i, (Gi, wi) in enumerate(shown)] \
        if c["op"] != "volume" else [(None, G)]
    Us, scale = _stored(c, U)
    return dict(c=c, g=g, G=G, f0=f0.to(_DT[c["storage"]]), mean=mean.to(_DT[c["storage"]]), U=Us,
                scale=scale, w=w, w0=w0, y=ys[0][0], frames=ys)


def prepare(case, seed):
    op = case["op"]
    if op == "pca":
        g = _grid(case)
        J, P, gen = case["J"], _patterns(g, min(5, case["K"] + 1), seed), _gen(seed + 9)
        d = torch.empty((J, 3) + g.shape, device="cuda")
        for j in range(J):
            t = 2.0 * math.pi * (j + 1) / (J + 1)
            co = ((1 - math.cos(t)) / 2, math.sin(t), (1 - math.cos(2 * t)) / 2, math.sin(2 * t),
                  (1 - math.cos(3 * t)) / 2)
            d[j] = sum(co[i] * P[i] for i in range(P.shape[0]))
            d[j] += 0.01 * torch.randn(d[j].shape, generator=gen, device="cuda")
        return dict(c=case, g=g, d=d)
    if op == "project":
        g, G = _grid(case), _geom(case)
        vol = _phantom(g, seed) + 1e-4 * torch.rand(g.shape, generator=_gen(seed + 3), device="cuda")
        return dict(c=case, g=g, G=G, vol=vol.to(_DT[case["compute"]]).contiguous())
    if op == "serve":
        srv = _lib.Server(64 << 30, max_slots=4, drop_stale=False)
        todo = []
        for i, c in enumerate(_streams(case)):
            s = _parts(c, seed * 100 + i, case["frames"])
            model = _lib.DeviceModel(s["mean"], s["U"], s["scale"])
            sid = srv.add_stream(s["g"], model, s["f0"], _opts(c, s["w"], s["w0"]), s["w0"])
            todo.append((sid, s["w0"], s["frames"]))
        return dict(c=case, srv=srv, todo=todo)
    s = _parts(case, seed)
    s["model"] = _lib.DeviceModel(s["mean"], s["U"], s["scale"])
    if op in ("solve", "cost_grad"):
        s["ctx"] = _lib.Context(s["g"], s["model"], s["f0"])
        s["opts"] = _opts(case, s["w"], s["w0"])
    if op == "autograd":
        s["w_t"] = torch.tensor(s["w0"], dtype=torch.float32, device="cuda", requires_grad=True)
        s["f0_t"] = s["f0"].clone().requires_grad_(True)
    return s


def run(state):
    c = state["c"]
    op = c["op"]
    if op == "solve":
        w, ab, st = state["ctx"].reconstruct(state["y"], state["G"], state["w0"], state["opts"])
        return dict(w=torch.tensor(w), ab=torch.tensor(ab), J=st["J"], tumour=torch.tensor(st["tumor_mm"]))
    if op == "cost_grad":
        J, grad = state["ctx"].cost_grad(state["y"], state["G"], state["w0"], _A, _B, c.get("mode", 0))
        return dict(J=J, grad=torch.tensor(grad))
    if op == "project":
        return _lib.forward_project(state["g"], state["G"], state["vol"])
    if op == "autograd":
        w, f0 = state["w_t"], state["f0_t"]
        p = autograd.project(w, f0, state["g"], state["G"], state["model"])
        gw, gf = torch.autograd.grad(((p - state["y"]) ** 2).sum(), (w, f0))
        return dict(p=p.detach(), grad_w=gw, grad_f0=gf)
    if op == "volume":
        x = _lib.dvf_compose(state["g"], state["model"], state["w"])
        return dict(dvf=x, f=_lib.warp_volume(state["g"], state["f0"], x))
    if op == "pca":
        mean, U, sing, wt = _lib.pca_train(state["g"], state["d"], c["K"])
        return dict(mean=mean, U=U, sing=sing, w_train=wt)
    srv = state["srv"]
    for sid, w0, frames in state["todo"]:
        srv.set_w(sid, w0)
        for y, G in frames:
            srv.submit(sid, y, G)
    srv.drain()
    done = sorted(srv.poll(1024), key=lambda r: r["req_id"])
    return dict(w=[torch.tensor(r["w"]) for r in done], J=torch.tensor([r["J"] for r in done]),
                tumour=torch.tensor([r["tumor_mm"] for r in done]))


# -------------------------------------------------------------- work -------
def _samples(c):
    """Samples that meet the box of the volume, from every 8th ray's chord."""
    g, G = _grid(c), _geom(c)
    st, ct = math.sin(G.angle), math.cos(G.angle)
    u = ((torch.arange(0, G.nu, 8) - 0.5 * (G.nu - 1)) * G.du)[None, :].double()
    v = ((torch.arange(0, G.nv, 8) - 0.5 * (G.nv - 1)) * G.dv)[:, None].double()
    s = (G.sad * st, -G.sad * ct, 0.0)
    d = (-G.sdd * st + u * ct + 0 * v, G.sdd * ct + u * st + 0 * v, v + 0 * u)
    L = (d[0] ** 2 + d[1] ** 2 + d[2] ** 2).sqrt()
    t0, t1 = torch.zeros_like(L), torch.ones_like(L)
    for a in range(3):
        h = 0.5 * g.fov[a]
        x = torch.where(d[a].abs() < 1e-9, torch.full_like(L, 1e-9), d[a])
        e = torch.stack([(-h - s[a]) / x, (h - s[a]) / x])
        t0, t1 = torch.maximum(t0, e.min(0)[0]), torch.minimum(t1, e.max(0)[0])
    return float(((t1 - t0).clamp(min=0) * L).mean()) / G.step * G.nu * G.nv


def work(case):
    """Inputs read once and outputs written once; the multiplications and
    additions of the trilinear sums (16 a channel and 27 a sample for position
    and weights), samples counted over the volume's box for a whole volume and
    over the body's share of it (0.4) for an evaluation of the model."""
    op = case["op"]
    if op == "serve":
        parts = [work(dict(s, frames=1)) for s in _streams(case)]
        return {k: case["frames"] * sum(p[k] for p in parts) for k in ("bytes", "flops")}
    N, M, K = case["nx"] * case["ny"] * case["nz"], case["nu"] * case["nv"], case["K"]
    sz, cs = _SIZE[case["storage"]], _SIZE[case["compute"]]
    warp = N * (60 + 30 * K)
    if op == "pca":
        J = case["J"]
        return dict(bytes=12.0 * N * (J + K + 1), flops=3.0 * N * (J * (J + 1) + 2 * J * (K + 1)))
    if op == "volume":
        return dict(bytes=float(N * (3 * (K + 1) * sz + sz + 12 + 4)), flops=float(N * (6 * K + 60)))
    n = _samples(case)
    if op == "project":
        return dict(bytes=float(cs * (N + M)), flops=43.0 * n)
    model = N * sz * (3 * (K + 1) + 1)
    if op == "autograd":
        return dict(bytes=float(model + 4 * N + 12 * M), flops=2 * 43.0 * n + 2.0 * warp)
    if op == "cost_grad" and case.get("mode", 0):
        return dict(bytes=float(model + 4 * M), flops=2 * 0.4 * 43.0 * n + 2.0 * warp)
    one = 0.4 * n * (27 + 16 * (K + 1)) + 0.5 * warp
    if op == "cost_grad":
        return dict(bytes=float(model + 4 * M), flops=one)
    return dict(bytes=9.0 * (model + 4 * M), flops=9.0 * one)   # nine evaluations a solve


# ------------------------------------------------------------- exact -------
def exact(case, seed):
    op = case["op"]
    if op in ("solve", "serve"):
        return None
    if op == "pca":
        s = prepare(case, seed)
        J, K, d = case["J"], case["K"], s["d"].view(case["J"], -1)
        mean = d.double().mean(0)
        E = [d[j].double() - mean for j in range(J)]
        G = torch.tensor([[float(E[i] @ E[j]) for j in range(J)] for i in range(J)], dtype=torch.float64)
        lam, V = torch.linalg.eigh(G)
        lam, V = lam.flip(0)[:K], V.flip(1)[:, :K]
        U = torch.stack([sum(float(V[j, k]) * E[j] for j in range(J)) / float(lam[k]) ** 0.5 for k in range(K)])
        sign = []
        for k in range(K):
            a = U[k].abs()
            i = int((a >= (1 - 1e-5) * a.max()).nonzero()[0])
            sign.append(-1.0 if float(U[k, i]) < 0 else 1.0)
            U[k] *= sign[k]
        shape = s["d"].shape[1:]
        wt = V * lam.sqrt() * torch.tensor(sign, dtype=torch.float64)
        return dict(mean=mean.view(shape), U=U.view((K,) + shape), sing=lam.sqrt().numpy(), w_train=wt.numpy())
    if op not in ("volume",) and _samples(case) > 4.0e8:
        return None                                  # over twenty seconds in 64 bits
    if op == "project":
        s = prepare(case, seed)
        return _project(s["g"], s["G"], s["vol"].double())
    s = _parts(case, seed)
    g, G = s["g"], s["G"]
    U = s["U"].double()
    if s["scale"]:
        U = U * torch.tensor(s["scale"], device="cuda", dtype=torch.float64).view(-1, 1, 1, 1, 1)
    mean, f0 = s["mean"].double(), s["f0"].double()
    if op == "volume":
        x = _compose(mean, U, s["w"])
        return dict(dvf=x, f=_interp(f0, _points(g, x)))
    w0 = torch.tensor(s["w0"], dtype=torch.float64)
    if op == "autograd":
        w0 = w0.float().double()
    w = w0.cuda().requires_grad_(True)
    f0.requires_grad_(op == "autograd")
    f = _interp(f0, _points(g, _compose(mean, U, w)))
    p = _project(g, G, f.detach())
    y = s["y"].double()
    r = p - y if op == "autograd" else p - _A * y - _B
    loss = (f * _backproject(g, G, 2.0 * r)).sum()
    if op == "autograd":
        gw, gf = torch.autograd.grad(loss, (w, f0))
        return dict(p=p, grad_w=gw, grad_f0=gf)
    return dict(J=float((r * r).sum()), grad=torch.autograd.grad(loss, w)[0])
