"""Far-field layer sums (csrc/far.hip) against the direct sums.

A composite call whose workspace lacks room for the far-field region takes the
direct route, so both routes run on the same inputs.  Each is within 1e-13 of
the exact sum relative to the largest term sum; the bar is the FP64 one,
1e-12 of the largest output."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _lattice(nv, sizes, seed):
    """nv ellipses in three rows of a channel, in random order."""
    rng = np.random.default_rng(seed)
    slot = rng.permutation(3 * -(-nv // 3))[:nv]
    xs, ys, off = [], [], [0]
    for i in range(nv):
        N = int(sizes[i % len(sizes)])
        t = 2 * np.pi * np.arange(N) / N
        p = rng.uniform(0.9, 2.2)
        ex, ey = 0.3 * np.cos(t), 0.14 * np.sin(t)
        xs.append(0.6 * (slot[i] // 3 + 0.5) + np.cos(p) * ex - np.sin(p) * ey)
        ys.append(0.68 * (slot[i] % 3 - 1.0) + np.sin(p) * ex + np.cos(p) * ey)
        off.append(off[-1] + N)
    return np.concatenate(xs), np.concatenate(ys), np.array(off, np.int32), 0.6 * -(-nv // 3)


def _close(a, b):
    import torch
    fa, fb = torch.isfinite(a), torch.isfinite(b)
    assert torch.equal(fa, fb)
    e = float((a[fa] - b[fb]).abs().max() / b[fb].abs().max())
    print(f"far against direct {e:.1e}", flush=True)
    assert e < 1e-12


# 61 x 96 = 5,856 nodes: just past the rule for three images; ragged sets, a
# last tile of two nodes; one image, which needs more nodes; one far image alone
@pytest.mark.parametrize("nv,sizes,img", [(61, (96,), (-1, 1)), (173, (50, 34, 66), (-1, 1)), (210, (50,), (0, 0)),
                                          (141, (64, 62), (-2, 1)), (105, (98,), (1, 1)), (300, (96,), (-1, 1))])
@pytest.mark.parametrize("mode", [0, 1])
def test_step_operator(nv, sizes, img, mode):
    import torch
    import paper_1510_05616_amd as s2d
    from paper_1510_05616_amd import vesicle as pv
    s2d.stokes2d_init(0)
    x, y, off, d = _lattice(nv, sizes, nv)
    V = pv.Vesicles(x, y, off)
    n = V.n
    z = torch.as_tensor(np.concatenate([np.cos(3 * x), np.sin(2 * y), 0.5 * np.cos(x) + 1.0]), device="cuda")
    p = pv.params(mode=mode, dt=1e-7, d=d, img_lo=img[0], img_hi=img[1])
    ws = V.workspace(p)
    print(f"step operator, {n} nodes, images {img}, mode {mode}", flush=True)
    out, _ = V.step_apply(p, z, with_rhs=False, ws=ws)
    again, _ = V.step_apply(p, z, with_rhs=False, ws=ws)
    p0 = pv.params(mode=0, dt=1e-7, d=d, img_lo=img[0], img_hi=img[1])
    direct, _ = V.step_apply(p0, z, with_rhs=False, ws=torch.empty(V.workspace(p0).numel() - 256, dtype=torch.uint8,
                                                                   device="cuda"))
    torch.cuda.synchronize()
    assert torch.equal(out, again)
    _close(out[:2 * n], direct[:2 * n])         # FP32C sums take the same FP64 far-field route


# 2 x 2,050 wall nodes refined 8 times = 32,800 sources; 8,193 targets: a last
# tile of one.  The targets hold outliers far along both axes, a coincident
# cluster and one NaN, which stays its own
@pytest.mark.parametrize("img", [(-1, 1), (0, 0)])
@pytest.mark.parametrize("accumulate", [0, 1])
def test_wall_correction(img, accumulate):
    import torch
    import synth
    import paper_1510_05616_amd as s2d
    from paper_1510_05616_amd import near as nr
    s2d.stokes2d_init(0)
    prob = synth.make_config(2, n_ves=1, wall_nodes=2050)
    walls = synth.wall_densities(prob.wall, 3)
    x, y = synth.near_wall_points(walls, 8193, 5)
    x[0], x[1], y[2] = 900.0, -40.0, 77.0
    x[100:230], y[100:230] = x[100], y[100]
    x[5000] = np.nan
    w, t = s2d.Curves(walls), s2d.Targets(x, y)
    need = nr.near_wall_workspace_size(w, t, 8)
    res = []
    print(f"wall correction, images {img}, accumulate {accumulate}", flush=True)
    for size in (need, need - 256):
        o = torch.full((2, t.n), 0.25, dtype=torch.float64, device="cuda")
        nr.near_wall_correct_eval(w, t, prob.d, img[0], img[1], 8, o[0], o[1], accumulate=accumulate,
                                  ws=torch.empty(size, dtype=torch.uint8, device="cuda"))
        res.append(o)
    torch.cuda.synchronize()
    assert torch.isnan(res[0][:, 5000]).all() and int(torch.isnan(res[0]).sum()) == 2
    _close(res[0], res[1])


def test_nan_source_reaches_every_target():
    import torch
    import paper_1510_05616_amd as s2d
    from paper_1510_05616_amd import vesicle as pv
    s2d.stokes2d_init(0)
    x, y, off, d = _lattice(100, (96,), 1)
    x[777] = np.nan
    V = pv.Vesicles(x, y, off)
    p = pv.params(dt=1e-7, d=d, img_lo=-1, img_hi=1)
    out, _ = V.step_apply(p, torch.ones(3 * V.n, dtype=torch.float64, device="cuda"), with_rhs=False)
    torch.cuda.synchronize()
    assert torch.isnan(out[:2 * V.n]).all()


def _mixed(seed, nv, sizes, n_free):
    """Vesicle curves with a density, targets at every second node in random
    order and n_free free points; curve 3 is made odd by dropping its last
    node, and a few on-curve entries are out of range."""
    import types
    from oracle import vesicle as ov
    x, y, off, d = _lattice(nv, sizes, seed)
    rng = np.random.default_rng(seed)
    keep = np.ones(len(x), bool)
    keep[off[4] - 1] = False
    g = ov.geometry(x, y, off)
    cut = off.copy()
    cut[4:] -= 1
    cs = types.SimpleNamespace(x=x[keep], y=y[keep], nx=g.nx[keep], ny=g.ny[keep], w=g.w[keep],
                               kappa=np.ones(keep.sum()), fx=rng.standard_normal(keep.sum()),
                               fy=rng.standard_normal(keep.sum()), curve_off=cut)
    node = rng.permutation(np.arange(0, keep.sum(), 2))
    curve = np.searchsorted(cut, node, side="right") - 1
    tx, ty = np.r_[cs.x[node], rng.uniform(0, d, n_free)], np.r_[cs.y[node], rng.uniform(1.1, 4.0, n_free)]
    oc = np.r_[curve, np.full(n_free, -1)].astype(np.int32)
    on = np.r_[node, np.full(n_free, -1)].astype(np.int32)
    return cs, tx, ty, oc, on, d


@pytest.mark.parametrize("op", [0, 1])
@pytest.mark.parametrize("mode,nv,sizes,n_free,img", [(0, 200, (58, 64), 1, (-1, 1)), (0, 330, (96, 46), 12001, (0, 0)),
                                                      (1, 330, (96, 46), 12001, (0, 0)), (1, 400, (62,), 3001, (0, 2))])
def test_eval_routes(op, mode, nv, sizes, n_free, img):
    import torch
    import oracle
    import paper_1510_05616_amd as s2d
    s2d.stokes2d_init(0)
    cs, tx, ty, oc, on, d = _mixed(7 + nv, nv, sizes, n_free)
    src = s2d.Curves(cs)
    bad = np.arange(5, 11)
    res = []
    print(f"op {op} mode {mode}: {src.n_nodes} sources, {len(tx)} targets, images {img}", flush=True)
    for wild in (False, True):
        c, k = oc.copy(), on.copy()
        if wild:
            c[bad[:3]], k[bad[3:]] = nv + 5, -7
        t = s2d.Targets(tx, ty, c, k)
        need = s2d.stokes2d_workspace_size(op, mode, src, t)
        for size in (need, need - 256):
            o = torch.zeros((2, t.n), dtype=torch.float64, device="cuda")
            ws = torch.empty(size, dtype=torch.uint8, device="cuda")
            m = mode if size == need else 0
            if op == 0:
                s2d.stokes2d_slp_eval(m, src, t, d, img[0], img[1], 0.7, o[0], o[1], 0, ws)
            else:
                s2d.stokes2d_dlp_eval(m, src, t, d, img[0], img[1], o[0], o[1], 0, ws)
            res.append(o)
    torch.cuda.synchronize()
    # the odd curve's targets (single layer) and the wild entries are NaN on both routes
    _close(res[0], res[1])
    assert torch.isnan(res[2][:, bad]).all()
    ok = np.setdiff1d(np.arange(len(tx)), bad)
    _close(res[2][:, ok], res[3][:, ok])
    idx = np.random.default_rng(1).choice(np.setdiff1d(ok, np.nonzero(oc == 3)[0]), 300, replace=False)
    if op == 0:
        ru, rv = oracle.slp(cs, tx[idx], ty[idx], oc[idx], on[idx], d, img[0], img[1], 0.7)
    else:
        ru, rv = oracle.dlp(cs, tx[idx], ty[idx], oc[idx], on[idx], d, img[0], img[1])
    g = res[0].cpu().numpy()[:, idx]
    e = np.hypot(g[0] - ru, g[1] - rv).max() / np.hypot(ru, rv).max()
    print(f"against the oracle {e:.1e}", flush=True)
    assert e < 1e-12


def test_capture_and_noalloc():
    """The far-field route recorded into a graph and replayed on changed
    densities with eager work between, and the no-allocation entry on the same
    route: bit for bit the eager call."""
    import torch
    import paper_1510_05616_amd as s2d
    s2d.stokes2d_init(0)
    cs, tx, ty, oc, on, d = _mixed(3, 240, (96,), 500)
    src, t = s2d.Curves(cs), s2d.Targets(tx, ty, oc, on)
    ws = torch.empty(s2d.stokes2d_workspace_size(0, 0, src, t), dtype=torch.uint8, device="cuda")
    o, e, q = (torch.zeros((2, t.n), dtype=torch.float64, device="cuda") for _ in range(3))
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        s2d.stokes2d_slp_eval(0, src, t, d, -1, 1, 1.0, o[0], o[1], 0, ws, st)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st):
            s2d.stokes2d_slp_eval(0, src, t, d, -1, 1, 1.0, o[0], o[1], 0, ws, st)
    for k in range(3):
        src.fx.mul_(1.5)
        g.replay()
        torch.cuda.synchronize()
        s2d.stokes2d_slp_eval(0, src, t, d, -1, 1, 1.0, e[0], e[1])
        s2d.stokes2d_slp_eval_noalloc(0, src, t, d, -1, 1, 1.0, q[0], q[1])
        torch.cuda.synchronize()
        assert torch.equal(o.nan_to_num(7.0), e.nan_to_num(7.0)) and torch.equal(q.nan_to_num(7.0), e.nan_to_num(7.0))


def test_noalloc_beyond_the_far_scratch():
    """500,000 sources: the far-field scratch does not fit the 32 MiB, the
    direct sum's does."""
    import torch
    import types
    import paper_1510_05616_amd as s2d
    s2d.stokes2d_init(0)
    n = 500_000
    rng = np.random.default_rng(0)
    a = lambda: rng.uniform(0, 1, n)
    src = s2d.Curves(types.SimpleNamespace(x=100 * a(), y=a(), nx=a(), ny=a(), w=a() / n, kappa=a(), fx=a(), fy=a(),
                                           curve_off=np.array([0, n], np.int32)))
    t = s2d.Targets(100 * rng.uniform(0, 1, 1100), 2.0 + rng.uniform(0, 1, 1100))
    far, direct = (torch.zeros((2, t.n), dtype=torch.float64, device="cuda") for _ in range(2))
    s2d.stokes2d_slp_eval(0, src, t, 100.0, -1, 1, 1.0, far[0], far[1])
    s2d.stokes2d_slp_eval_noalloc(0, src, t, 100.0, -1, 1, 1.0, direct[0], direct[1])
    torch.cuda.synchronize()
    assert not torch.equal(far, direct)
    _close(far, direct)


@pytest.mark.parametrize("mode,nv,sizes,n_free,img", [(0, 120, (62, 64), 9001, (-1, 1)), (1, 300, (96, 50), 9001, (-1, 1)),
                                                      (0, 200, (96,), 12001, (1, 1))])
def test_pressure_and_traction_routes(mode, nv, sizes, n_free, img):
    import torch
    import oracle
    import paper_1510_05616_amd as s2d
    s2d.stokes2d_init(0)
    cs, tx, ty, oc, on, d = _mixed(nv, nv, sizes, n_free)
    tx, ty = tx[-n_free:], ty[-n_free:]
    src, t = s2d.Curves(cs), s2d.Targets(tx, ty)
    ang = np.random.default_rng(2).uniform(0, 2 * np.pi, n_free)
    nx, ny = (torch.as_tensor(f(ang), device="cuda") for f in (np.cos, np.sin))
    idx = np.random.default_rng(3).choice(n_free, 200, replace=False)
    print(f"mode {mode}: {src.n_nodes} sources, {n_free} targets, images {img}", flush=True)

    def run(op, m, size):
        o = torch.full((2, t.n), 0.5, dtype=torch.float64, device="cuda")
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        if op == s2d.S2D_OP_SLP_PRESSURE:
            s2d.stokes2d_slp_pressure_eval(m, src, t, d, img[0], img[1], o[0], 1, ws)
        elif op == s2d.S2D_OP_DLP_PRESSURE:
            s2d.stokes2d_dlp_pressure_eval(m, src, t, d, img[0], img[1], 0.7, o[0], 1, ws)
        else:
            s2d.stokes2d_slp_traction_eval(m, src, t, nx, ny, d, img[0], img[1], o[0], o[1], 1, ws)
        torch.cuda.synchronize()
        return o - 0.5

    refs = {s2d.S2D_OP_SLP_PRESSURE: lambda: (oracle.slp_pressure(cs, tx[idx], ty[idx], d, img[0], img[1]),),
            s2d.S2D_OP_DLP_PRESSURE: lambda: (oracle.dlp_pressure(cs, tx[idx], ty[idx], d, img[0], img[1], 0.7),),
            s2d.S2D_OP_SLP_TRACTION: lambda: oracle.slp_traction(cs, tx[idx], ty[idx], np.cos(ang[idx]), np.sin(ang[idx]),
                                                                 d, img[0], img[1])}
    for op, ref in refs.items():
        need = s2d.stokes2d_workspace_size(op, mode, src, t)
        far, direct = run(op, mode, need), run(op, 0, need - 256)
        if op != s2d.S2D_OP_SLP_TRACTION:
            assert torch.equal(far[1], torch.zeros_like(far[1]))
        _close(far, direct)
        r = np.array(ref())
        e = np.abs(far.cpu().numpy()[:len(r), idx] - r).max() / np.abs(r).max()
        print(f"op {op} against the oracle {e:.1e}", flush=True)
        assert e < 1e-12


# A target that is not finite keeps that to itself, wherever its tile lies
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_targets_that_are_not_finite(bad):
    import torch
    import types
    import paper_1510_05616_amd as s2d
    s2d.stokes2d_init(0)
    x, y, off, d = _lattice(100, (96,), 3)
    rng = np.random.default_rng(8)
    c = types.SimpleNamespace(x=x, y=y, nx=np.cos(x), ny=np.sin(x), w=np.full(len(x), 1e-2), kappa=None,
                              fx=rng.standard_normal(len(x)), fy=rng.standard_normal(len(x)), curve_off=off)
    src = s2d.Curves(c)
    tx, ty = rng.uniform(0, d, 9000), rng.uniform(1.0, 1.4, 9000)
    ref, out = (torch.zeros(4, 9000, dtype=torch.float64, device="cuda") for _ in range(2))
    k = np.array([7, 4000, 4001, 8999])
    for o in (ref, out):
        t = s2d.Targets(tx, ty)
        s2d.stokes2d_slp_eval(0, src, t, d, -1, 1, 1.0, o[0], o[1])
        s2d.stokes2d_dlp_eval(0, src, t, d, -1, 1, o[2], o[3])
        tx[k[:2]] = bad
        ty[k[1:]] = bad
    torch.cuda.synchronize()
    rest = torch.ones(9000, dtype=torch.bool, device="cuda")
    rest[k] = False
    assert not torch.isfinite(out[:, ~rest]).any()
    _close(out[:, rest], ref[:, rest])


def _time(f):
    import torch
    f()
    best = float("inf")
    for _ in range(5):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(4):
            f()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / 4)
    return best


# A few points far outside the others (placeholder coordinates) must not take
# the sort keys' resolution from them: the sum stays right everywhere and costs
# their own tiles, here 3 of 450 (every pair near would cost thirty times the
# sum; the bar leaves a factor of two for the clock).  Target outliers on either
# axis, at 1e3 and 1e30 channel lengths, infinite (any number of those); a source
# outlier.
@pytest.mark.parametrize("where", ["target x", "target y", "huge", "inf", "many inf", "nan", "source"])
def test_outliers_keep_the_rest_far(where):
    import torch
    import types
    import paper_1510_05616_amd as s2d
    s2d.stokes2d_init(0)
    x, y, off, d = _lattice(300, (96,), 11)
    rng = np.random.default_rng(4)
    c = types.SimpleNamespace(x=x, y=y, nx=np.cos(x), ny=np.sin(x), w=np.full(len(x), 1e-2), kappa=None,
                              fx=rng.standard_normal(len(x)), fy=rng.standard_normal(len(x)), curve_off=off)
    tx, ty = rng.uniform(0, d, len(x)), rng.uniform(1.0, 1.4, len(x))
    base = s2d.Curves(c), s2d.Targets(tx, ty)
    k = [7, 15000, 28000] if where != "many inf" else np.arange(20000, 23000)
    if where == "source":
        c.x = x.copy()
        c.x[k] = 3e3 * d
    elif where == "target y":
        ty = ty.copy()
        ty[k] = -1e3 * d
    else:
        tx = tx.copy()
        tx[k] = {"target x": 1e3 * d, "huge": 1e30 * d, "nan": np.nan}.get(where, np.inf)
        tx[k[1:]] *= -1             # among the first tiles in the sort order, too
    src, trg = s2d.Curves(c), s2d.Targets(tx, ty)
    out = torch.zeros(2, len(x), dtype=torch.float64, device="cuda")
    ws = torch.empty(s2d.stokes2d_workspace_size(0, 0, src, trg), dtype=torch.uint8, device="cuda")
    plain = _time(lambda: s2d.stokes2d_slp_eval(0, *base, d, -1, 1, 1.0, out[0], out[1], 0, ws))
    t = _time(lambda: s2d.stokes2d_slp_eval(0, src, trg, d, -1, 1, 1.0, out[0], out[1], 0, ws))
    print(f"{where}: {t:.3f} ms, without outliers {plain:.3f}", flush=True)
    ref = torch.zeros_like(out)
    # the direct sum of the same targets, 1,000 at a time (fewer than the far route takes)
    for i in range(0, len(x), 1000):
        s2d.stokes2d_slp_eval(0, src, s2d.Targets(tx[i:i + 1000], ty[i:i + 1000]), d, -1, 1, 1.0, ref[0, i:i + 1000],
                              ref[1, i:i + 1000])
    torch.cuda.synchronize()
    fa, fb = torch.isfinite(out), torch.isfinite(ref)
    assert torch.equal(fa, fb)
    near = torch.ones(len(x), dtype=torch.bool, device="cuda")
    near[k] = False
    for sel in (near, ~near):
        a, b, f = out[:, sel], ref[:, sel], fa[:, sel]
        if f.any():
            e = float((a[f] - b[f]).abs().max() / b[f].abs().max())
            print(f"{where}: far against direct {e:.1e}", flush=True)
            assert e < 1e-12
    assert t < 2 * plain


# The route taken with the queried workspace is no slower than the direct sums
# of the same call (a workspace that holds no more than those), by a bar that
# leaves the clock a tenth: few targets against many sources, and pressures,
# whose direct terms are the cheapest, on both sides of the line.
@pytest.mark.parametrize("op,mode,ns,nt", [(0, 1, 256000, 1100), (0, 1, 2880, 30000), (2, 0, 2880, 30000),
                                           (4, 0, 2400, 30000), (2, 1, 9984, 9000), (2, 0, 20160, 20000),
                                           (1, 0, 9984, 14000)])
def test_route_is_the_faster_one(op, mode, ns, nt):
    import torch
    import types
    import paper_1510_05616_amd as s2d
    s2d.stokes2d_init(0)
    x, y, off, d = _lattice(ns // 96, (96,), 5)
    rng = np.random.default_rng(2)
    c = types.SimpleNamespace(x=x, y=y, nx=np.cos(x), ny=np.sin(x), w=np.full(len(x), 1e-2), kappa=None,
                              fx=rng.standard_normal(len(x)), fy=rng.standard_normal(len(x)), curve_off=off)
    src, trg = s2d.Curves(c), s2d.Targets(rng.uniform(0, d, nt), rng.uniform(-1.2, 1.2, nt))
    u = torch.zeros(4, nt, dtype=torch.float64, device="cuda")
    full = s2d.stokes2d_workspace_size(op, mode, src, trg)

    def call(ws):
        if op == 0:
            s2d.stokes2d_slp_eval(mode, src, trg, d, -1, 1, 1.0, u[0], u[1], 0, ws)
        elif op == 1:
            s2d.stokes2d_dlp_eval(mode, src, trg, d, -1, 1, u[0], u[1], 0, ws)
        elif op == 2:
            s2d.stokes2d_slp_pressure_eval(mode, src, trg, d, -1, 1, u[0], 0, ws)
        else:
            s2d.stokes2d_slp_traction_eval(mode, src, trg, u[2], u[3], d, -1, 1, u[0], u[1], 0, ws)

    ws = torch.empty(full, dtype=torch.uint8, device="cuda")
    # the least workspace that the call takes is the direct plan's
    lo, hi = 256, full
    while hi - lo > 4096:
        mid = (lo + hi) // 2 // 256 * 256
        try:
            call(ws[:mid])
            hi = mid
        except s2d.S2DError:
            lo = mid
    direct = min(_time(lambda: call(ws[:hi])) for _ in range(2))
    t = min(_time(lambda: call(ws)) for _ in range(2))
    print(f"operator {op} mode {mode}, {ns} x {nt}: {t:.3f} ms, direct {direct:.3f}", flush=True)
    assert t < 1.1 * direct


# The far-field sums are FP64 in either mode, so FP32C has nothing to refine:
# the same solve, sum for sum (25 sums against 20 on 96,000 nodes before)
@pytest.mark.parametrize("warm,near", [(0, 0), (1, 0), (0, 1)])
def test_step_solve_is_the_same_in_both_modes(warm, near):
    import torch
    import paper_1510_05616_amd as s2d
    from paper_1510_05616_amd import vesicle as pv
    s2d.stokes2d_init(0)
    x, y, off, d = _lattice(75, (96,), 21)
    V = pv.Vesicles(x, y, off)
    L0, A0 = V.measure()
    res = []
    for mode in (0, 1):
        W = pv.Vesicles(x, y, off)
        p = pv.params(mode=mode, dt=1e-4, d=d, img_lo=-1, img_hi=1, L0=L0, tol=1e-10, nmax=96, near=near, near_P=4,
                      near_band=4.0, warm=warm)
        uv = [torch.full((V.n,), 1e-3, dtype=torch.float64, device="cuda") for _ in range(2)]
        it = W.time_step(p, A0=A0, uv=uv)
        res.append((W.x, W.y, W.sigma, *uv, it))
    torch.cuda.synchronize()
    print(f"warm {warm}, near {near}: iterations and residual {res[0][-1]}, {res[1][-1]}", flush=True)
    assert res[0][-1] == res[1][-1] and res[0][-1][1] <= 1e-10
    for a, b in zip(res[0][:-1], res[1][:-1]):
        assert torch.equal(a, b)
