"""The calls whose time matters to a user of this library, over the sizes that
its configurations, tests and benchmark have.

A case is a dict of plain values; `prepare` builds what a program holds before
the call (device arrays, workspaces, a factored cell, a packed network), `run`
is one pass through the public entry points, `exact` the same quantities in
plain 64-bit torch, `work` the bytes and operations a pass cannot do without.

FP64-mode results are returned as the library's FP64 arrays.  FP32C-mode
results carry FP32 accuracy (the library states 1e-6), and the program that
asks for that mode keeps them as float32: `run` returns that array.
"""
import math
import types

import numpy as np
import torch

import paper_1510_05616_amd as s2d
from paper_1510_05616_amd import near as nr
from paper_1510_05616_amd import vesicle as pv
from paper_1510_05616_amd.cell import Cell

DEV = "cuda"
F64 = torch.float64
MODES = {"f64": s2d.S2D_FP64, "f32c": s2d.S2D_FP32C}
_ready = False


def _init():
    global _ready
    if not _ready:
        s2d.stokes2d_init(0)
        _ready = True


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # the smallest channel (configuration 1): one vesicle of 64 nodes, 256
        # nodes per wall; one interaction evaluation, where launches count
        dict(name="step_small_f64", kind="step", mode="f64", nv=1, nn=64, nw=256, ns=0, ragged=False),
        # configuration 2: 50 vesicles, a mid-size channel, the FP32C mode
        dict(name="step_mid_f32c", kind="step", mode="f32c", nv=50, nn=128, nw=2048, ns=0, ragged=False),
        # the 128k-node channel (configuration 3), the benchmark's workload, in
        # both modes: 1,000 vesicles of 96 nodes, 2 x 16,000 wall nodes, 64
        # side targets
        dict(name="step_channel_f32c", kind="step", mode="f32c", nv=1000, nn=96, nw=16000, ns=32, ragged=False),
        dict(name="step_channel_f64", kind="step", mode="f64", nv=1000, nn=96, nw=16000, ns=32, ragged=False),
        # pressure and traction fields at scattered points of a channel with
        # vesicles of mixed node counts (visualisation, stress data)
        dict(name="fields_f32c", kind="fields", mode="f32c", nv=300, nn=96, nw=4500, nt=30011, ragged=True),
        # many small channels at once (configuration 4's batched call)
        dict(name="batch_f32c", kind="batch", mode="f32c", ni=64, nv_max=40, nw_max=4096),
        # close evaluation by upsampled quadrature: an odd number of targets
        # near curves of 64-128 nodes (labels, reference, fallback)
        dict(name="near_quad", kind="near_quad", nt=100003, P=8),
        # configuration 5's inference: 1e6 near targets, per-curve tolerances
        dict(name="near_auto", kind="near_auto", nt=1000000, tol=1e-5),
        # training of the near-field network: minibatches of 1,024, forward,
        # backward and Adam
        dict(name="near_train", kind="near_train", nt=50000, batch=1024, steps=50),
        # close evaluation of the walls' double layer at near-wall targets
        dict(name="wall_near", kind="wall_near", nw=16000, nt=20000, P=8),
        # the channel's response to its vesicles (Algorithm 1, steps 3-5)
        dict(name="response", kind="response", mode="f64", nv=240, nn=96, nw=2000, K=32, M=128),
        # one time step (Algorithm 1, steps 6-9) of the channel's vesicles
        # with close evaluation between near vesicles
        dict(name="time_step", kind="time_step", mode="f64", nv=1000, nn=96, ragged=False, near=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 5 + ["fields"] * 2 + ["batch", "near_quad", "near_auto", "near_train", "wall_near",
                                                      "response", "response", "time_step", "time_step"])
    mode = rng.choice(["f64", "f32c"])
    ragged = rng.random() < 0.5
    if kind == "step":
        return dict(kind=kind, mode=mode, nv=_log(rng, 1, 1000), nn=2 * rng.randint(16, 48), nw=_log(rng, 200, 16000),
                    ns=rng.choice([0, 16, 32]), ragged=ragged)
    if kind == "fields":
        return dict(kind=kind, mode=mode, nv=_log(rng, 1, 300), nn=2 * rng.randint(16, 48), nw=_log(rng, 200, 4500),
                    nt=_log(rng, 60, 30000), ragged=ragged)
    if kind == "batch":
        return dict(kind=kind, mode=mode, ni=_log(rng, 2, 64), nv_max=rng.randint(1, 40), nw_max=_log(rng, 300, 4096))
    if kind == "near_quad":
        return dict(kind=kind, nt=_log(rng, 200, 100000), P=rng.choice([4, 8]))
    if kind == "near_auto":
        return dict(kind=kind, nt=_log(rng, 1000, 1000000), tol=rng.choice([1e-5, 3e-5, 1e-4]))
    if kind == "near_train":
        return dict(kind=kind, nt=_log(rng, 5000, 50000), batch=rng.choice([256, 1000, 1024]), steps=rng.randint(5, 50))
    if kind == "wall_near":
        return dict(kind=kind, nw=2 * _log(rng, 200, 8000), nt=_log(rng, 100, 20000), P=rng.choice([4, 8]))
    if kind == "response":
        return dict(kind=kind, mode="f64", nv=_log(rng, 1, 240), nn=2 * rng.randint(16, 48), nw=2 * _log(rng, 100, 1000),
                    K=rng.choice([16, 32]), M=rng.choice([64, 128]))
    return dict(kind=kind, mode="f64", nv=_log(rng, 2, 1000), nn=2 * rng.randint(16, 48), ragged=ragged,
                near=rng.random() < 0.5)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _ellipses(cx, cy, a, b, phi, sizes, fx=None, fy=None):
    """Curve arrays of ellipses (one entry per curve) with `sizes` nodes each."""
    off = np.zeros(len(sizes) + 1, np.int64)
    off[1:] = np.cumsum(sizes)
    c = np.repeat(np.arange(len(sizes)), sizes)
    t = 2 * np.pi * (np.arange(off[-1]) - off[c]) / sizes[c]
    ct, st, cp, sp = np.cos(t), np.sin(t), np.cos(phi)[c], np.sin(phi)[c]
    A, B = a[c], b[c]
    x = cx[c] + cp * A * ct - sp * B * st
    y = cy[c] + sp * A * ct + cp * B * st
    xp, yp = -cp * A * st - sp * B * ct, -sp * A * st + cp * B * ct
    v = np.hypot(xp, yp)
    o = types.SimpleNamespace(x=x, y=y, nx=yp / v, ny=-xp / v, w=2 * np.pi / sizes[c] * v, kappa=A * B / v ** 3,
                              curve_off=off.astype(np.int32), curve=c, t=t, fx=fx, fy=fy)
    return o


def _density(rng, o, K):
    """Per curve and component sum_k k^-2 (a_k cos k t + b_k sin k t)."""
    nc = len(o.curve_off) - 1
    out = []
    for _ in range(2):
        f = np.zeros_like(o.t)
        ab = rng.standard_normal((K, 2, nc))
        for k in range(1, K + 1):
            f += (ab[k - 1, 0][o.curve] * np.cos(k * o.t) + ab[k - 1, 1][o.curve] * np.sin(k * o.t)) / (k * k)
        out.append(f)
    o.fx, o.fy = out
    return o


def _profile(d):
    """Half-height of the wavy channel of period d and its derivatives."""
    s = 2 * math.pi * max(1, round(d / (2 * math.pi))) / d
    return (lambda x: 1.5 + 0.4 * np.sin(s * x) + 0.2 * np.sin(3 * s * x),
            lambda x: s * (0.4 * np.cos(s * x) + 0.6 * np.cos(3 * s * x)),
            lambda x: -s * s * (0.4 * np.sin(s * x) + 1.8 * np.sin(3 * s * x)))


def _walls(rng, d, nw, K):
    h, hp, hpp = _profile(d)
    xs = d * np.arange(nw) / nw
    sp = np.sqrt(1 + hp(xs) ** 2)
    cat = np.concatenate
    o = types.SimpleNamespace(
        x=cat([xs, xs]), y=cat([h(xs), -h(xs)]), nx=cat([-hp(xs) / sp, -hp(xs) / sp]), ny=cat([1 / sp, -1 / sp]),
        w=cat([d / nw * sp] * 2), kappa=cat([-hpp(xs) / sp ** 3] * 2),
        curve_off=np.array([0, nw, 2 * nw], np.int32), curve=np.repeat([0, 1], nw), t=cat([2 * np.pi * xs / d] * 2))
    return _density(rng, o, K) if K else o


def _vesicles(rng, nv, nn, ragged, K):
    """nv vesicles (reduced areas 0.65-0.9, one area) on a jittered three-row
    lattice of the channel, in random order; returns the curves and the
    period.  Node counts depend on (nv, nn) alone."""
    cols = max(11, -(-nv // 3))
    d = 0.6 * cols
    slot = rng.permutation(3 * cols)[:nv]
    ratio = rng.uniform(0.37, 0.62, nv)
    a = np.sqrt(0.12064 / math.pi / ratio)
    pick = np.random.default_rng([nv, nn]).choice([max(16, 2 * (nn // 3)), nn, 2 * (2 * nn // 3)], nv)
    sizes = (pick if ragged else np.full(nv, nn)).astype(np.int64)
    o = _ellipses(0.6 * (slot // 3 + 0.5) + rng.uniform(-0.04, 0.04, nv), 0.68 * (slot % 3 - 1.0), a, a * ratio,
                  math.pi / 2 + rng.uniform(-0.5, 0.5, nv), sizes)
    return _density(rng, o, K), d


def _f64(n, *shape):
    return torch.empty((n,) + shape, dtype=F64, device=DEV)


def _refs(o, at, n):
    """on_curve / on_node of n targets whose entries from `at` on are o's nodes."""
    c, k = np.full(n, -1, np.int32), np.full(n, -1, np.int32)
    m = len(o.x)
    c[at:at + m] = o.curve
    k[at:at + m] = np.arange(m)
    return c, k


def _channel(rng, case):
    ves, d = _vesicles(rng, case["nv"], case["nn"], case["ragged"], 8)
    wall = _walls(rng, d, case["nw"], 8)
    return ves, wall, d


def _step_data(rng, case):
    ves, wall, d = _channel(rng, case)
    ns = case["ns"]
    ys = _profile(d)[0](0.0) * np.polynomial.legendre.leggauss(ns)[0] if ns else np.zeros(0)
    x = np.concatenate([ves.x, wall.x, np.zeros(ns), np.full(ns, d)])
    y = np.concatenate([ves.y, wall.y, ys, ys])
    n = len(x)
    return ves, wall, d, x, y, _refs(ves, 0, n), _refs(wall, len(ves.x), n)


def _near_set(rng, nt):
    """Ellipses of 64-128 nodes, about 200 targets each at log-uniform normal
    distances of 0.05 to 5 mean spacings (configuration 5)."""
    nc = (nt + 199) // 200
    ratio = rng.uniform(0.37, 0.62, nc)
    a = np.sqrt(math.pi * 0.3 * 0.17 / math.pi / ratio)
    sizes = np.random.default_rng(nc).choice([64, 96, 128], nc).astype(np.int64)
    phi = rng.uniform(0, math.pi, nc)
    z = np.zeros(nc)
    o = _density(rng, _ellipses(z, z, a, a * ratio, phi, sizes), 12)
    h = np.add.reduceat(o.w, o.curve_off[:-1]) / sizes
    tc = np.minimum(np.arange(nt) // 200, nc - 1)
    th = rng.uniform(0, 2 * math.pi, nt)
    A, B, cp, sp = a[tc], (a * ratio)[tc], np.cos(phi)[tc], np.sin(phi)[tc]
    ex, ey, dx, dy = A * np.cos(th), B * np.sin(th), -A * np.sin(th), B * np.cos(th)
    qx, qy = cp * dx - sp * dy, sp * dx + cp * dy
    v = np.hypot(qx, qy)
    de = h[tc] * 10.0 ** rng.uniform(math.log10(0.05), math.log10(5.0), nt)
    return o, cp * ex - sp * ey + de * qy / v, sp * ex + cp * ey - de * qx / v, tc.astype(np.int32)


def _dev(o):
    return s2d.Curves(o, DEV)


def prepare(case, seed):
    _init()
    rng = np.random.default_rng([int(seed), 17])
    kind = case["kind"]
    s = types.SimpleNamespace(kind=kind, mode=MODES.get(case.get("mode")), f32=case.get("mode") == "f32c", mu=1.0)
    if kind == "step":
        ves, wall, s.d, x, y, rv, rw = _step_data(rng, case)
        s.ves, s.wall = _dev(ves), _dev(wall)
        s.tv, s.tw = s2d.Targets(x, y, *rv, device=DEV), s2d.Targets(x, y, *rw, device=DEV)
        s.out = _f64(2, len(x))
        s.ws = [torch.empty(s2d.stokes2d_workspace_size(op, s.mode, a, b), dtype=torch.uint8, device=DEV)
                for op, a, b in ((s2d.S2D_OP_SLP, s.ves, s.tv), (s2d.S2D_OP_DLP, s.wall, s.tw))]
    elif kind == "fields":
        ves, wall, s.d = _channel(rng, case)
        s.ves, s.wall = _dev(ves), _dev(wall)
        x, y, ang = _field_points(rng, case, s.d)
        s.trg = s2d.Targets(x, y, device=DEV)
        s.nx, s.ny = (torch.as_tensor(f(ang), dtype=F64, device=DEV) for f in (np.cos, np.sin))
        s.out = _f64(3, len(x))
        s.ws = torch.empty(max(s2d.stokes2d_workspace_size(op, s.mode, a, s.trg) for op, a in (
            (s2d.S2D_OP_SLP_PRESSURE, s.ves), (s2d.S2D_OP_DLP_PRESSURE, s.wall), (s2d.S2D_OP_SLP_TRACTION, s.ves))),
            dtype=torch.uint8, device=DEV)
    elif kind == "batch":
        s.inst, s.out, s.keep = [], None, []
        data = _batch_data(rng, case)
        s.out = _f64(2, sum(len(q[3]) for q in data))
        at = 0
        for ves, wall, d, x, y, rv, rw in data:
            n = len(x)
            s.inst.append(s2d.BatchInstance(_dev(ves), _dev(wall), s2d.Targets(x, y, *rv, device=DEV),
                                            s2d.Targets(x, y, *rw, device=DEV), d, 1.0, s.out[0, at:at + n],
                                            s.out[1, at:at + n]))
            at += n
        s.ws = torch.empty(s2d.stokes2d_batch_workspace_size(s.mode, s.inst), dtype=torch.uint8, device=DEV)
    elif kind in ("near_quad", "near_auto", "near_train"):
        o, x, y, tc = _near_set(rng, case["nt"])
        if kind == "near_train":
            _prepare_train(s, case, seed, o, x, y, tc)
            return s
        s.P = case.get("P", 8)
        s.ves, s.trg = _dev(o), s2d.Targets(x, y, device=DEV)
        s.tc = torch.as_tensor(tc, device=DEV)
        s.out = _f64(2, len(x))
        s.method, s.blob, s.tol, s.used = nr.S2D_NEAR_UPSAMPLE, None, None, None
        if kind == "near_auto":
            s.method = nr.S2D_NEAR_AUTO
            s.blob, s.tol = _network(seed, o, x, y, tc, case["tol"])
            s.used = torch.empty(len(x), dtype=torch.int32, device=DEV)
        s.ws = torch.empty(nr.near_workspace_size(s.method, s.ves, s.trg, s.P), dtype=torch.uint8, device=DEV)
    elif kind == "wall_near":
        wall, s.d, x, y = _wall_data(rng, case)
        s.P = case["P"]
        s.wall, s.trg = _dev(wall), s2d.Targets(x, y, device=DEV)
        s.out = _f64(2, len(x))
        s.ws = torch.empty(nr.near_wall_workspace_size(s.wall, s.trg, s.P), dtype=torch.uint8, device=DEV)
    elif kind == "response":
        ves, s.d = _vesicles(rng, case["nv"], case["nn"], False, 4)
        wall = _walls(rng, s.d, case["nw"], 0)
        sy = _profile(s.d)[0](0.0) * np.polynomial.legendre.leggauss(case["K"])[0]
        s.cell = Cell(wall, sy, s.d, case["M"], s.mu, device=DEV)
        s.cell.factor()
        s.V = pv.Vesicles(ves.x, ves.y, ves.curve_off, device=DEV)
        s.fx, s.fy = (torch.as_tensor(v, dtype=F64, device=DEV) for v in (ves.fx, ves.fy))
    elif kind == "time_step":
        ves, s.d = _vesicles(rng, case["nv"], case["nn"], case["ragged"], 1)
        s.V = pv.Vesicles(ves.x, ves.y, ves.curve_off, device=DEV)
        s.x0, s.y0 = s.V.x.clone(), s.V.y.clone()
        nmax = int(np.diff(ves.curve_off).max())
        s.L0, s.A0 = s.V.measure()
        s.p = pv.params(mode=s.mode, dt=1e-4, kappa_b=1.0, mu=s.mu, d=s.d, img_lo=-1, img_hi=1, L0=s.L0, tol=1e-10,
                        nmax=nmax, near=int(case["near"]), near_P=8, near_band=5.0, near_max=1 << 20)
        s.uv = (_f64(s.V.n), _f64(s.V.n))
        s.ws = s.V.workspace(s.p)
    else:
        raise ValueError(kind)
    return s


def _field_points(rng, case, d):
    """Points of the fluid between the vesicle rows and the walls, with the
    angles of their normals."""
    n = case["nt"]
    x = rng.uniform(0, d, n)
    top = _profile(d)[0](x)
    y = np.where(rng.random(n) < 0.5, 1.0 + rng.uniform(0.05, 0.95, n) * (top - 1.0 - 0.02), 0.34)
    y = np.where(top - 0.02 < y, 0.34, y) * np.where(rng.random(n) < 0.5, 1.0, -1.0)
    return x, y, rng.uniform(0, 2 * math.pi, n)


def _batch_data(rng, case):
    out, size = [], np.random.default_rng([case["ni"], case["nv_max"], case["nw_max"]])
    for _ in range(case["ni"]):
        c = dict(nv=int(size.integers(1, case["nv_max"] + 1)), nn=int(size.choice([32, 64, 128])), ragged=True,
                 nw=int(size.integers(min(256, case["nw_max"]), case["nw_max"] + 1)), ns=0)
        out.append(_step_data(rng, c))
    return out


def _wall_data(rng, case):
    """Wall nodes moved 0.05 to 3 spacings into the channel."""
    d = 64 * math.pi * case["nw"] / 16000
    wall = _walls(rng, d, case["nw"], 5)
    n = case["nt"]
    i = rng.integers(0, 2 * case["nw"], n)
    a, b = rng.uniform(0.05, 3.0, n) * wall.w[i], rng.uniform(-0.5, 0.5, n) * wall.w[i]
    return wall, d, wall.x[i] - a * wall.nx[i] - b * wall.ny[i], wall.y[i] - a * wall.ny[i] + b * wall.nx[i]


def _standardised(seed, X):
    """Network parameters: seeded weights, the input standardisation of X."""
    p = torch.as_tensor(nr.init_weights(int(seed) % (1 << 31)).astype(np.float32), device=DEV)
    nr.near_feature_stats(X, p)
    return p


def _network(seed, o, x, y, tc, tol):
    """A packed network with seeded weights and bounds of the calibrated
    tables' form (errors and corrections decaying like exp(-2 pi b), no
    learned route past the nodes' midpoint), and the per-curve tolerances."""
    m = min(len(x), 20000)
    data = nr.NearData(o, x[:m], y[:m], tc[:m], labels=False, device=DEV)
    p = _standardised(seed, data.X)
    b = 10.0 ** (nr.BIN_LO + nr.BIN_W * np.arange(nr.N_BINS))
    zero = np.repeat(3.0 * np.exp(-2 * math.pi * b), nr.CELL)
    err = 1e-3 * np.repeat(np.exp(-2 * math.pi * b), nr.CELL).reshape(nr.N_BINS, nr.S_BINS, nr.K_BINS)
    err *= (1.0 + np.arange(nr.S_BINS))[None, :, None] * (0.5 + 0.25 * np.arange(nr.K_BINS))[None, None, :]
    err[:, -1, :] = 3e38
    f32 = dict(dtype=torch.float32, device=DEV)
    blob = torch.zeros(nr.near_mlp_blob_size(), dtype=torch.uint8, device=DEV)
    nr.near_mlp_pack(p, torch.as_tensor(err.reshape(-1), **f32), nr.N_BINS, nr.BIN_LO, nr.BIN_W, blob,
                     bound_zero=torch.as_tensor(zero, **f32))
    return blob, torch.full((len(o.curve_off) - 1,), 0.2 * tol, dtype=F64, device=DEV)


def _prepare_train(s, case, seed, o, x, y, tc):
    s.data = nr.NearData(o, x, y, tc, device=DEV)
    s.batch, s.steps = case["batch"], case["steps"]
    s.p0 = _standardised(seed, s.data.X)
    g = torch.Generator(device="cpu")
    g.manual_seed(int(seed))
    pool = torch.nonzero((s.data.b >= 0.04) & (s.data.T[:, 12] > 0)).view(-1).to(torch.int32)
    pick = torch.randint(0, pool.numel(), (s.steps, s.batch), generator=g).to(DEV)
    s.idx = pool[pick.view(-1)].view(s.steps, s.batch)
    s.par, s.m, s.v, s.grad = (torch.zeros_like(s.p0) for _ in range(4))
    s.loss = torch.zeros(1, dtype=torch.float32, device=DEV)
    s.ws = torch.empty(nr.near_mlp_train_workspace_size(s.batch), dtype=torch.uint8, device=DEV)


TRAIN_LR = 1e-5      # the low end of the training schedule's rates


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(s):
    k = s.kind
    if k == "step":
        # u = S f + D tau at every node (Algorithm 1's interactions)
        u, v = s.out[0], s.out[1]
        s2d.stokes2d_slp_eval(s.mode, s.ves, s.tv, s.d, -1, 1, s.mu, u, v, 0, s.ws[0])
        s2d.stokes2d_dlp_eval(s.mode, s.wall, s.tw, s.d, -1, 1, u, v, 1, s.ws[1])
    elif k == "fields":
        s2d.stokes2d_slp_pressure_eval(s.mode, s.ves, s.trg, s.d, -1, 1, s.out[0], 0, s.ws)
        s2d.stokes2d_dlp_pressure_eval(s.mode, s.wall, s.trg, s.d, -1, 1, s.mu, s.out[0], 1, s.ws)
        s2d.stokes2d_slp_traction_eval(s.mode, s.ves, s.trg, s.nx, s.ny, s.d, -1, 1, s.out[1], s.out[2], 0, s.ws)
    elif k == "batch":
        s2d.stokes2d_batch_eval(s.mode, s.inst, s.ws)
    elif k == "near_quad" or k == "near_auto":
        nr.near_correct_eval(s.method, s.ves, s.trg, s.tc, s.P, s.blob, 0.0, s.mu, s.out[0], s.out[1], s.used, s.ws,
                             curve_tol=s.tol)
        if s.used is not None:
            return s.out, s.used
    elif k == "near_train":
        s.par.copy_(s.p0)
        s.m.zero_()
        s.v.zero_()
        for j in range(s.steps):
            nr.near_mlp_train_step(s.batch, s.idx[j], s.data.X, s.data.T, s.par, s.m, s.v, j + 1, TRAIN_LR, s.grad,
                                   s.loss, s.ws)
        return s.par, s.grad, s.loss
    elif k == "wall_near":
        nr.near_wall_correct_eval(s.wall, s.trg, s.d, -1, 1, s.P, s.out[0], s.out[1], ws=s.ws)
    elif k == "response":
        return s.V.channel_response(s.cell, s.fx, s.fy, 10.0, s.mode)
    elif k == "time_step":
        s.V.x.copy_(s.x0)
        s.V.y.copy_(s.y0)
        s.V.sigma.zero_()
        s.V.time_step(s.p, A0=s.A0, ws=s.ws, uv=s.uv)
        return s.V.x, s.V.y, s.V.sigma, s.uv[0], s.uv[1]
    return s.out.float() if s.f32 else s.out


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def _sizes(case):
    """Expected vesicle nodes of a case (ragged sets vary by seed)."""
    return case["nv"] * case["nn"]


def work(case):
    """Bytes: each input and output once (a source node 48-64 bytes, a target
    16-32 in and 16 out).  Operations: 19 a pair and image for the layers'
    velocities and the traction, 11 and 18 for the two pressures (a logarithm
    or reciprocal counted as one)."""
    k = case["kind"]
    if k == "step":
        ns, nw = _sizes(case), 2 * case["nw"]
        nt = ns + nw + 2 * case["ns"]
        return {"bytes": 64.0 * (ns + nw) + 40.0 * nt, "flops": 19.0 * 3 * nt * (ns + nw)}
    if k == "fields":
        ns, nw, nt = _sizes(case), 2 * case["nw"], case["nt"]
        return {"bytes": 48.0 * (2 * ns + nw) + 80.0 * nt, "flops": 3.0 * nt * (30 * ns + 18 * nw)}
    if k == "batch":
        n = [len(q[3]) for q in _batch_data(np.random.default_rng(0), case)]
        return {"bytes": 104.0 * sum(n), "flops": 57.0 * sum(m * m for m in n)}
    if k == "near_quad":
        nt, n = case["nt"], 96.0
        return {"bytes": nt * (36.0 + n * 40 / 200), "flops": nt * n * 19.0 * (case["P"] + 1)}
    if k == "near_auto":
        # about half the targets through the network (2 x 10,500 operations)
        # and a quarter through the quadrature
        nt, n = case["nt"], 96.0
        return {"bytes": nt * (40.0 + n * 72 / 200), "flops": nt * (0.5 * 21000 + 0.25 * n * 19.0 * 9)}
    if k == "near_train":
        return {"bytes": case["steps"] * (case["batch"] * 116.0 + 10580 * 24.0),
                "flops": case["steps"] * case["batch"] * 6.0 * 10368}
    if k == "wall_near":
        n, nt = 2.0 * case["nw"], case["nt"]
        return {"bytes": 64.0 * n + 32.0 * nt, "flops": 57.0 * nt * n * (case["P"] + 1)}
    if k == "response":
        ns, nw = _sizes(case), 2.0 * case["nw"]
        n = 2 * nw
        return {"bytes": 8.0 * n * n + 64.0 * (ns + nw), "flops": 2 * 57.0 * ns * nw + 2.0 * n * n + 19.0 * ns * case["M"]}
    # time step: about 20 operator evaluations, the preconditioner's blocks
    # factored once and applied each time
    ns, m = _sizes(case), 3.0 * case["nn"]
    return {"bytes": 20 * case["nv"] * 8.0 * m * m, "flops": 20 * 57.0 * ns * ns + case["nv"] * (2 / 3 * m ** 3 + 40 * m * m)}


# ---------------------------------------------------------------------------
# 64-bit values
# ---------------------------------------------------------------------------
def _t(v):
    return torch.as_tensor(v, dtype=F64, device=DEV)


def _kress(N):
    """T_j, j = 0..N-1: Kress's weights for log(4 sin^2(t/2)) as the own-curve
    coefficient of w_k f_k (T_0 without the speed term)."""
    m = N // 2
    j = np.arange(N)
    p = np.arange(1, m)[:, None]
    T = (np.cos(2 * np.pi * ((p * j) % N) / N) / p).sum(0) + np.where(j % 2, -1.0, 1.0) / N
    T[1:] += np.log(2 * np.abs(np.sin(np.pi * j[1:] / N)))
    return T


CHUNK = 1 << 27      # (target, source) pairs of one block of the direct sums


def _direct(term, x, y, src, d, images, comps):
    """sum over images and sources of term(rx, ry, q, own) at every target."""
    n, m = len(x), len(src)
    out = torch.zeros((comps, n), dtype=F64, device=DEV)
    step = max(1, min(n, CHUNK // max(1, m)))
    for i in range(0, n, step):
        X, Y = x[i:i + step, None], y[i:i + step, None]
        for k in images:
            rx = X - (src[None, :, 0] + k * d) if k else X - src[None, :, 0]
            ry = Y - src[None, :, 1]
            term(out[:, i:i + step], rx, ry, rx * rx + ry * ry, k, i)
    return out


def _exact_slp(o, x, y, curve, d, images):
    """Single layer without 1 / (4 pi mu); curve: per target its own curve or -1."""
    g = torch.stack([_t(o.w * o.fx), _t(o.w * o.fy)])
    oc, own = _t(o.curve).to(torch.int32), _t(curve).to(torch.int32)

    def term(out, rx, ry, q, k, i):
        lq, iq = torch.log(q).mul_(-0.5), 1.0 / q
        if k == 0:
            same = own[i:i + rx.shape[0], None] == oc[None, :]
            lq.masked_fill_(same, 0.0)
            iq.masked_fill_(same, 0.0)
        out += g @ lq.T
        a, b, c = rx * rx * iq, rx * ry * iq, ry * ry * iq
        out[0] += a @ g[0] + b @ g[1]
        out[1] += b @ g[0] + c @ g[1]

    return _direct(term, _t(x), _t(y), torch.stack([_t(o.x), _t(o.y)], 1), d, images, 2)


def _exact_self(o):
    """Own-curve part at the nodes of o, Kress's rule, without 1 / (4 pi mu)."""
    out = np.zeros((2, len(o.x)))
    for N in np.unique(np.diff(o.curve_off)):
        N = int(N)
        lo = o.curve_off[:-1][np.diff(o.curve_off) == N]
        T = _kress(N)
        ii = (np.arange(N)[:, None] - np.arange(N)[None, :]) % N
        for part in np.array_split(lo, max(1, len(lo) * N * N // (1 << 23))):
            at = part[:, None] + np.arange(N)
            X, Y, W, NX, NY = (a[at] for a in (o.x, o.y, o.w, o.nx, o.ny))
            gx, gy = W * o.fx[at], W * o.fy[at]
            rx, ry = X[:, :, None] - X[:, None, :], Y[:, :, None] - Y[:, None, :]
            q = rx * rx + ry * ry
            e = np.arange(N)
            q[:, e, e] = 1.0
            L = T[ii][None] - 0.5 * np.log(q)
            L[:, e, e] = T[0] - np.log(W * N / (2 * math.pi))
            axx, axy, ayy = rx * rx / q, rx * ry / q, ry * ry / q
            axx[:, e, e], axy[:, e, e], ayy[:, e, e] = 1 - NX * NX, -NX * NY, 1 - NY * NY
            out[0, at] = np.einsum("cij,cj->ci", L + axx, gx) + np.einsum("cij,cj->ci", axy, gy)
            out[1, at] = np.einsum("cij,cj->ci", axy, gx) + np.einsum("cij,cj->ci", L + ayy, gy)
    return out


def _exact_dlp(o, x, y, node, d, images):
    """Double layer without 1 / pi; node: per target its own node or -1."""
    nx, ny, tx, ty = _t(o.w * o.nx), _t(o.w * o.ny), _t(o.fx), _t(o.fy)
    nd = _t(node).to(torch.int64)

    def term(out, rx, ry, q, k, i):
        f = (rx * nx + ry * ny).mul_(rx * tx + ry * ty).div_(q * q)
        if k == 0:
            r = nd[i:i + rx.shape[0]]
            at = torch.nonzero(r >= 0).view(-1)
            f[at, r[at]] = 0.0
        out[0] += (f * rx).sum(1)
        out[1] += (f * ry).sum(1)

    out = _direct(term, _t(x), _t(y), torch.stack([_t(o.x), _t(o.y)], 1), d, images, 2)
    at = np.nonzero(node >= 0)[0]
    j = node[at]
    c = -0.5 * o.kappa[j] * o.w[j]
    tn = o.nx[j] * o.fx[j] + o.ny[j] * o.fy[j]
    out[0, at] += _t(c * (o.fx[j] - o.nx[j] * tn))
    out[1, at] += _t(c * (o.fy[j] - o.ny[j] * tn))
    return out


def _exact_step(ves, wall, d, x, y, rv, rw):
    s = _exact_slp(ves, x, y, rv[0], d, (-1, 0, 1))
    s[:, :len(ves.x)] += _t(_exact_self(ves))
    return s / (4 * math.pi) + _exact_dlp(wall, x, y, rw[1], d, (-1, 0, 1)) / math.pi


def _exact_fields(rng, case):
    ves, wall, d = _channel(rng, case)
    x, y, ang = _field_points(rng, case, d)
    X, Y = _t(x), _t(y)
    gx, gy = _t(ves.w * ves.fx), _t(ves.w * ves.fy)
    mx, my = _t(np.cos(ang))[:, None], _t(np.sin(ang))[:, None]
    nx, ny, tx, ty = _t(wall.w * wall.nx), _t(wall.w * wall.ny), _t(wall.fx), _t(wall.fy)

    def single(out, rx, ry, q, k, i):
        rg = (rx * gx + ry * gy).div_(q)
        out[0] += rg.sum(1) / (2 * math.pi)
        n = rx.shape[0]
        f = rg * (rx * mx[i:i + n] + ry * my[i:i + n]) / q / -math.pi
        out[1] += (f * rx).sum(1)
        out[2] += (f * ry).sum(1)

    def double(out, rx, ry, q, k, i):
        f = 2 * (rx * nx + ry * ny) * (rx * tx + ry * ty) / (q * q) - (nx * tx + ny * ty) / q
        out[0] += f.sum(1) / math.pi

    a = _direct(single, X, Y, torch.stack([_t(ves.x), _t(ves.y)], 1), d, (-1, 0, 1), 3)
    return a + _direct(double, X, Y, torch.stack([_t(wall.x), _t(wall.y)], 1), d, (-1, 0, 1), 3)


def _refine(v, P):
    """Trigonometric interpolation of the rows of v onto P times the nodes,
    the Nyquist mode split evenly, and its derivative."""
    N = v.shape[-1]
    V = np.fft.fft(v)
    W = np.zeros(v.shape[:-1] + (P * N,), complex)
    h = N // 2
    W[..., :h], W[..., -h + 1:] = V[..., :h], V[..., h + 1:]
    W[..., h] += 0.5 * V[..., h]
    W[..., P * N - h] += 0.5 * V[..., h]
    m = np.fft.fftfreq(P * N, 1.0 / (P * N))
    return np.fft.ifft(W).real * P, np.fft.ifft(1j * m * W).real * P


def _exact_near(rng, case):
    o, x, y, tc = _near_set(rng, case["nt"])
    P = case["P"]
    out = torch.zeros((2, len(x)), dtype=F64, device=DEV)
    sizes = np.diff(o.curve_off)
    for N in np.unique(sizes):
        N = int(N)
        cs = np.nonzero(sizes == N)[0]
        at = o.curve_off[cs][:, None] + np.arange(N)
        (X, dX), (Y, dY), (FX, _), (FY, _) = (_refine(a[at], P) for a in (o.x, o.y, o.fx, o.fy))
        W = 2 * math.pi / (P * N) * np.hypot(dX, dY)
        rows = np.concatenate([np.stack([X, Y, W * FX, W * FY]),
                               np.stack([o.x[at], o.y[at], -o.w[at] * o.fx[at], -o.w[at] * o.fy[at]])], -1)
        rows = _t(rows)
        where = np.full(len(sizes), -1)
        where[cs] = np.arange(len(cs))
        ti = np.nonzero(where[tc] >= 0)[0]
        for part in np.array_split(ti, max(1, len(ti) * rows.shape[-1] // (1 << 26))):
            sx, sy, gx, gy = rows[:, torch.as_tensor(where[tc[part]], device=DEV)]
            rx, ry = _t(x[part])[:, None] - sx, _t(y[part])[:, None] - sy
            q = rx * rx + ry * ry
            lq, t = -0.5 * torch.log(q), (rx * gx + ry * gy) / q
            p = torch.as_tensor(part, device=DEV)
            out[0, p] = (lq * gx + rx * t).sum(1)
            out[1, p] = (lq * gy + ry * t).sum(1)
    return out / (4 * math.pi)


def _exact_wall(rng, case):
    wall, d, x, y = _wall_data(rng, case)
    P, nw = case["P"], case["nw"]
    t = 2 * math.pi * np.arange(nw) / nw
    tf = 2 * math.pi * np.arange(P * nw) / (P * nw)
    parts = []
    for c in range(2):
        s = slice(c * nw, (c + 1) * nw)
        X, dX = _refine(wall.x[s] - d * t / (2 * math.pi), P)
        Y, dY = _refine(wall.y[s], P)
        X, dX = X + d * tf / (2 * math.pi), dX + d / (2 * math.pi)
        v = np.hypot(dX, dY)
        sg = 1.0 if c == 0 else -1.0
        parts.append((X, Y, -sg * dY / v, sg * dX / v, 2 * math.pi / (P * nw) * v, _refine(wall.fx[s], P)[0],
                      _refine(wall.fy[s], P)[0]))
    f = [np.concatenate(q) for q in zip(*parts)]
    fine = types.SimpleNamespace(**dict(zip(("x", "y", "nx", "ny", "w", "fx", "fy"), f)), kappa=np.zeros(2 * P * nw))
    free = np.full(len(x), -1)
    return (_exact_dlp(fine, x, y, free, d, (-1, 0, 1)) - _exact_dlp(wall, x, y, free, d, (-1, 0, 1))) / math.pi


def _exact_train(case, seed):
    """The Adam steps in 64-bit torch from the same records."""
    s = prepare(case, seed)
    par, mean, sd = s.p0.double(), s.p0[:14].double(), s.p0[14:28].double()
    m, v = torch.zeros_like(par), torch.zeros_like(par)
    X, T = s.data.X.double(), s.data.T.double()
    for j in range(s.steps):
        p = par.clone().requires_grad_(True)
        w = {k: p[nr.OFF[k]:nr.OFF[k] + int(np.prod(sh))].view(sh) for k, sh in nr.SHAPES.items()}
        i = s.idx[j].long()
        h, r = (X[i] - mean) / sd, T[i]
        for k in "123":
            h = torch.nn.functional.gelu(h @ w["W" + k] + w["b" + k], approximate="tanh")
        c = (h @ w["W4"] + w["b4"]).view(-1, 5, 2, 2)
        e = r[:, 12:13] * (r[:, 13:14] * (c * r[:, :10].view(-1, 5, 1, 2)).sum((1, 3)) - r[:, 10:12])
        loss = 0.5 * (e * e).sum() / s.batch
        g, = torch.autograd.grad(loss, p)
        g[:28] = 0.0
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        par = par - TRAIN_LR * (m / (1 - 0.9 ** (j + 1))) / ((v / (1 - 0.999 ** (j + 1))).sqrt() + 1e-8)
    return par, g, loss.detach().view(1)


def exact(case, seed):
    """None for the learned route (its network runs in BF16 by design), the
    channel response (a truncated pseudo-inverse) and the time step (GMRES to
    a tolerance)."""
    _init()
    rng = np.random.default_rng([int(seed), 17])
    k = case["kind"]
    if k == "step":
        return _exact_step(*_step_data(rng, case))
    if k == "fields":
        return _exact_fields(rng, case)
    if k == "batch":
        return torch.cat([_exact_step(*q) for q in _batch_data(rng, case)], 1)
    if k == "near_quad":
        return _exact_near(rng, case)
    if k == "near_train":
        return _exact_train(case, seed)
    if k == "wall_near":
        return _exact_wall(rng, case) if case["nw"] * case["nt"] * case["P"] <= 3e9 else None
    return None
