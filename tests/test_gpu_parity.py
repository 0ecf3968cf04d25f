"""GPU parity: the HIP path through the C ABI against the FP64 oracle, element
by element on the same seeded inputs.

Tolerances (relative error E of Section 5, per target class and per part):
FP64 mode 1e-12, FP32C mode 1e-6.  Full-size (config 3, 128,064 targets x
128,000 sources x 3 images) runs the GPU on every target in the same launch
configuration the benchmark times, and checks a seeded sample of targets that
the oracle computes one by one.
"""
import numpy as np
import pytest

import synth
from _common import class_errors, gpu_eval, oracle_eval, rel_err, sample_targets

pytestmark = pytest.mark.gpu

TOL = {0: 1e-12, 1: 1e-6}
MODES = [0, 1]


@pytest.fixture(scope="module", autouse=True)
def device():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1510_05616_amd as s2d
    s2d.stokes2d_init(0)
    yield


def _check(prob, mode, idx=None, img=(-1, 1), tol=None):
    tol = TOL[mode] if tol is None else tol
    g = gpu_eval(prob, mode, *img, idx=idx)
    o = oracle_eval(prob, *img, idx=idx)
    kind = prob.trg.kind if idx is None else prob.trg.kind[idx]
    errs = {}
    for part, (gu, gv, ou, ov) in (("slp", (g[0], g[1], o[0], o[1])), ("dlp", (g[2], g[3], o[2], o[3]))):
        for cls, e in class_errors(kind, gu, gv, ou, ov).items():
            errs[f"{part}/{cls}"] = e
    tot = class_errors(kind, g[0] + g[2], g[1] + g[3], o[0] + o[2], o[1] + o[3])
    for cls, e in tot.items():
        errs[f"total/{cls}"] = e
    worst = max(errs.values())
    print(f"mode={mode} worst E={worst:.3e} {errs}", flush=True)
    assert worst <= tol, errs
    return errs


@pytest.mark.parametrize("mode", MODES)
def test_config1_parity(mode):
    _check(synth.make_config(1), mode)


@pytest.mark.parametrize("mode", MODES)
def test_config2_parity(mode):
    _check(synth.make_config(2), mode)


@pytest.fixture(scope="module")
def cfg3():
    return synth.make_config(3)


@pytest.mark.parametrize("mode", MODES)
def test_config3_full_size_sampled(cfg3, mode):
    idx = sample_targets(cfg3, per_class=256, seed=5)
    _check(cfg3, mode, idx=idx)


@pytest.mark.parametrize("img", [(0, 0), (1, 1), (-1, -1), (-2, 2), (-3, 0)])
@pytest.mark.parametrize("mode", MODES)
def test_image_ranges(mode, img):
    _check(synth.make_config(1), mode, img=img)


@pytest.mark.parametrize("mode", MODES)
def test_ragged_sizes(mode):
    # sizes that are not multiples of the wave (64), the target tile or the
    # source superblock (256); odd wall node count
    prob = synth.make_config(2, n_ves=7, ves_nodes=38, wall_nodes=1001)
    _check(prob, mode)


def _translated(prob, dx, dy):
    import dataclasses
    move = lambda cs: dataclasses.replace(cs, x=cs.x + dx, y=cs.y + dy)
    trg = dataclasses.replace(prob.trg, x=prob.trg.x + dx, y=prob.trg.y + dy)
    return dataclasses.replace(prob, ves=move(prob.ves), wall=move(prob.wall), trg=trg)


@pytest.mark.parametrize("mode", MODES)
def test_translated_channel(mode):
    """The whole channel moved far from the origin. FP32C forms differences
    against FP64 origins per tile, so its error must not grow with the
    coordinates' magnitude; both sides see the same translated inputs."""
    _check(_translated(synth.make_config(2), 3.0e3, -7.0e2), mode)


@pytest.mark.parametrize("mode", MODES)
def test_near_touching_vesicles(mode):
    """Vesicle 1 moved towards vesicle 0 until their nearest nodes are a fifth
    of a node spacing apart (the near sub-blocks of FP32C, r formed in FP64)."""
    import dataclasses
    prob = synth.make_config(2)
    v, off = prob.ves, prob.ves.curve_off
    s0, s1 = slice(off[0], off[1]), slice(off[1], off[2])
    x0, y0, x1, y1 = v.x[s0], v.y[s0], v.x[s1], v.y[s1]
    h = np.sum(v.w[s0]) / (off[1] - off[0])
    ux, uy = x0.mean() - x1.mean(), y0.mean() - y1.mean()
    gap = lambda a: np.sqrt(((x0[:, None] - (x1[None, :] + a * ux)) ** 2 +
                             (y0[:, None] - (y1[None, :] + a * uy)) ** 2).min())
    # the first approach to 0.2 h along the line of centres: scan, then bisect
    steps = np.linspace(0.0, 1.0, 401)
    k = int(np.argmax([gap(a) < 0.2 * h for a in steps]))
    assert k > 0
    lo, hi = steps[k - 1], steps[k]
    for _ in range(60):
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if gap(mid) > 0.2 * h else (lo, mid)
    sx, sy = lo * ux, lo * uy
    x, y = v.x.copy(), v.y.copy()
    x[s1] += sx
    y[s1] += sy
    tx, ty = prob.trg.x.copy(), prob.trg.y.copy()
    on1 = prob.trg.ves_curve == 1
    tx[on1] += sx
    ty[on1] += sy
    prob = dataclasses.replace(prob, ves=dataclasses.replace(v, x=x, y=y),
                               trg=dataclasses.replace(prob.trg, x=tx, y=ty))
    print(f"nearest node gap {gap(lo) / h:.3f} h", flush=True)
    _check(prob, mode)


def test_single_node_sources_and_free_targets():
    import torch
    import oracle
    import paper_1510_05616_amd as s2d
    rng = np.random.default_rng(9)
    src = synth.concat_curves([(rng.normal(size=1), rng.normal(size=1), np.ones(1), np.zeros(1),
                                np.ones(1), np.zeros(1), rng.normal(size=1), rng.normal(size=1))
                               for _ in range(3)])
    tx, ty = rng.normal(size=5) + 5.0, rng.normal(size=5)
    c, tg = s2d.Curves(src), s2d.Targets(tx, ty)
    for mode in MODES:
        u = torch.zeros(5, dtype=torch.float64, device="cuda")
        v = torch.zeros_like(u)
        s2d.stokes2d_slp_eval(mode, c, tg, 3.0, -1, 1, 0.7, u, v)
        ou, ov = oracle.slp(src, tx, ty, d=3.0, img_lo=-1, img_hi=1, mu=0.7)
        assert rel_err(u.cpu().numpy(), v.cpu().numpy(), ou, ov) < TOL[mode]
        s2d.stokes2d_dlp_eval(mode, c, tg, 3.0, -1, 1, u, v)
        ou, ov = oracle.dlp(src, tx, ty, d=3.0, img_lo=-1, img_hi=1)
        assert rel_err(u.cpu().numpy(), v.cpu().numpy(), ou, ov) < TOL[mode]


def test_empty_inputs_and_accumulate():
    import torch
    import paper_1510_05616_amd as s2d
    prob = synth.make_config(1)
    t = prob.trg
    ves = s2d.Curves(prob.ves)
    tv = s2d.Targets(t.x, t.y, t.ves_curve, t.ves_node)
    # no targets: a no-op
    e = s2d.Targets(np.zeros(0), np.zeros(0))
    z = torch.zeros(0, dtype=torch.float64, device="cuda")
    s2d.stokes2d_slp_eval(0, ves, e, prob.d, -1, 1, 1.0, z, z)
    # no sources: zero output; with accumulate the outputs are unchanged
    empty = synth.concat_curves([])
    ec = s2d.Curves(empty)
    tf = s2d.Targets(t.x, t.y)
    u = torch.full((t.n,), 3.5, dtype=torch.float64, device="cuda")
    v = torch.full((t.n,), -1.5, dtype=torch.float64, device="cuda")
    s2d.stokes2d_slp_eval(0, ec, tf, prob.d, -1, 1, 1.0, u, v, accumulate=1)
    torch.cuda.synchronize()
    assert torch.all(u == 3.5) and torch.all(v == -1.5)
    s2d.stokes2d_dlp_eval(1, ec, tf, prob.d, -1, 1, u, v)
    torch.cuda.synchronize()
    assert torch.all(u == 0) and torch.all(v == 0)
    # accumulate adds exactly the non-accumulated result
    for mode in MODES:
        a = torch.zeros(t.n, dtype=torch.float64, device="cuda")
        b = torch.zeros_like(a)
        s2d.stokes2d_slp_eval(mode, ves, tv, prob.d, -1, 1, 1.0, a, b)
        u = torch.full((t.n,), 0.25, dtype=torch.float64, device="cuda")
        v = torch.full((t.n,), -0.5, dtype=torch.float64, device="cuda")
        s2d.stokes2d_slp_eval(mode, ves, tv, prob.d, -1, 1, 1.0, u, v, accumulate=1)
        torch.cuda.synchronize()
        assert torch.equal(u, a + 0.25) and torch.equal(v, b - 0.5)


def test_inconsistent_on_curve_entries_give_nan():
    import torch
    import paper_1510_05616_amd as s2d
    prob = synth.make_config(1)
    t = prob.trg
    vc, vn = t.ves_curve.copy(), t.ves_node.copy()
    vn[3] = vn[3] + 200                 # node outside its curve
    vc[5] = 7                           # curve that does not exist
    wc, wn = t.wall_curve.copy(), t.wall_node.copy()
    j = int(np.where(wc >= 0)[0][0])
    wn[j] = -5
    ves, wall = s2d.Curves(prob.ves), s2d.Curves(prob.wall)
    for mode in MODES:
        u = torch.zeros(t.n, dtype=torch.float64, device="cuda")
        v = torch.zeros_like(u)
        s2d.stokes2d_slp_eval(mode, ves, s2d.Targets(t.x, t.y, vc, vn), prob.d, -1, 1, 1.0, u, v)
        un = u.cpu().numpy()
        assert np.isnan(un[3]) and np.isnan(un[5])
        assert np.isfinite(np.delete(un, [3, 5])).all()
        s2d.stokes2d_dlp_eval(mode, wall, s2d.Targets(t.x, t.y, wc, wn), prob.d, -1, 1, u, v)
        un = u.cpu().numpy()
        assert np.isnan(un[j]) and np.isfinite(np.delete(un, [j])).all()


def test_odd_curve_with_self_target_gives_nan():
    import torch
    import paper_1510_05616_amd as s2d
    c = synth.ellipse_curve(0.3, 0.2, 33, fx=np.cos, fy=np.sin)
    oc = np.zeros(33, np.int32)
    on = np.arange(33, dtype=np.int32)
    u = torch.zeros(33, dtype=torch.float64, device="cuda")
    v = torch.zeros_like(u)
    s2d.stokes2d_slp_eval(0, s2d.Curves(c), s2d.Targets(c.x, c.y, oc, on), 0.0, 0, 0, 1.0, u, v)
    assert torch.isnan(u).all()


@pytest.mark.parametrize("mode", MODES)
def test_bitwise_deterministic(mode):
    prob = synth.make_config(2)
    a = gpu_eval(prob, mode)
    b = gpu_eval(prob, mode)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


def test_workspace_errors():
    import torch
    import paper_1510_05616_amd as s2d
    prob = synth.make_config(1)
    t = prob.trg
    ves = s2d.Curves(prob.ves)
    tv = s2d.Targets(t.x, t.y, t.ves_curve, t.ves_node)
    u = torch.zeros(t.n, dtype=torch.float64, device="cuda")
    v = torch.zeros_like(u)
    need = s2d.stokes2d_workspace_size(0, 0, ves, tv)
    small = torch.empty(need // 2, dtype=torch.uint8, device="cuda")
    with pytest.raises(s2d.S2DError) as ei:
        s2d.stokes2d_slp_eval(0, ves, tv, prob.d, -1, 1, 1.0, u, v, ws=small)
    assert ei.value.code == s2d.S2D_EWORKSPACE
    big = torch.empty(need + 512, dtype=torch.uint8, device="cuda")
    with pytest.raises(s2d.S2DError) as ei:   # misaligned pointer
        s2d.stokes2d_slp_eval(0, ves, tv, prob.d, -1, 1, 1.0, u, v, ws=big[8:])
    assert ei.value.code == s2d.S2D_EWORKSPACE


@pytest.mark.parametrize("mode", MODES)
def test_side_targets_few_targets_many_sources(cfg3, mode):
    # only the 64 side-wall collocation points of the 128k workload: one target
    # tile against every source superblock, so the call splits the sources over
    # hundreds of waves and reduces the partials in a second pass
    import torch
    import oracle
    import paper_1510_05616_amd as s2d
    t = cfg3.trg
    side = np.where(t.kind == 2)[0]
    tx, ty = t.x[side], t.y[side]
    ves, wall = s2d.Curves(cfg3.ves), s2d.Curves(cfg3.wall)
    tg = s2d.Targets(tx, ty)
    for img in ((-1, 1), (1, 1), (-1, -1)):
        u = torch.zeros(len(side), dtype=torch.float64, device="cuda")
        v = torch.zeros_like(u)
        s2d.stokes2d_slp_eval(mode, ves, tg, cfg3.d, img[0], img[1], cfg3.mu, u, v)
        ou, ov = oracle.slp(cfg3.ves, tx, ty, None, None, cfg3.d, img[0], img[1], cfg3.mu)
        e1 = rel_err(u.cpu().numpy(), v.cpu().numpy(), ou, ov)
        s2d.stokes2d_dlp_eval(mode, wall, tg, cfg3.d, img[0], img[1], u, v)
        ou, ov = oracle.dlp(cfg3.wall, tx, ty, None, None, cfg3.d, img[0], img[1])
        e2 = rel_err(u.cpu().numpy(), v.cpu().numpy(), ou, ov)
        print(f"side targets mode={mode} images={img}: slp {e1:.2e} dlp {e2:.2e}", flush=True)
        assert e1 <= TOL[mode] and e2 <= TOL[mode]


# launch shapes of the direct sums: superblocks of 16 sources (the first three),
# of 64 and of 256 with one and more split groups, groups chosen for full rounds
# of the chip; counts around the tile (64), the superblocks and their records.
# One far image alone in FP64 only: the sums of a few float terms at one distance
# cancel to a tenth of the terms and less.
@pytest.mark.parametrize("n_ves,ves_nodes,wall_nodes", [(1, 10, 9), (1, 16, 65), (3, 64, 257), (10, 66, 515),
                                                        (20, 64, 1000), (40, 96, 1025), (60, 64, 1500)])
@pytest.mark.parametrize("img,mode", [((-1, 1), 0), ((-1, 1), 1), ((0, 0), 0), ((0, 0), 1), ((1, 1), 0)])
def test_direct_launch_shapes(n_ves, ves_nodes, wall_nodes, img, mode):
    prob = synth.make_config(2, n_ves=n_ves, ves_nodes=ves_nodes, wall_nodes=wall_nodes)
    errs = _check(prob, mode, idx=sample_targets(prob, per_class=256, seed=3), img=img)
    if n_ves == 1 and img == (0, 0):
        # a lone vesicle's own nodes have Kress's rule only, in FP64 in either mode
        assert errs["slp/vesicle"] <= 1e-13


# A layer applied in place: the outputs are the density, so Kress's rule on a
# curve of many tiles (2,046 nodes: 32, the last one ragged) must not meet
# another tile's results.  The kernels' order of summation is the same: same bits.
@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("sizes", [(2046,), (130, 64, 258), (34,)])
def test_single_layer_in_place(sizes, mode):
    import torch
    import paper_1510_05616_amd as s2d
    cs = synth.concat_curves([tuple(getattr(c, k) for k in ("x", "y", "nx", "ny", "w", "kappa", "fx", "fy"))
                              for c in (synth.ellipse_curve(0.3, 0.2, n, (1.1 * i, 0.0), fx=np.cos, fy=np.sin)
                                        for i, n in enumerate(sizes))])
    oc = np.repeat(np.arange(len(sizes), dtype=np.int32), sizes)
    on = np.arange(sum(sizes), dtype=np.int32)
    src, t = s2d.Curves(cs), s2d.Targets(cs.x, cs.y, oc, on)
    want = torch.zeros(2, t.n, dtype=torch.float64, device="cuda")
    s2d.stokes2d_slp_eval(mode, src, t, 9.0, -1, 1, 1.3, want[0], want[1])
    s2d.stokes2d_slp_eval(mode, src, t, 9.0, -1, 1, 1.3, src.fx, src.fy)
    torch.cuda.synchronize()
    assert torch.equal(src.fx, want[0]) and torch.equal(src.fy, want[1])


# Without sources every on-curve reference is out of range: NaN with the
# workspace the size query names, and a call without one is refused.
@pytest.mark.parametrize("mode", MODES)
def test_no_sources_with_on_curve_targets(mode):
    import torch
    import paper_1510_05616_amd as s2d
    n = 1000
    oc = np.where(np.arange(n) % 3 == 0, 0, -1).astype(np.int32)
    src = s2d.Curves(synth.concat_curves([]))
    t = s2d.Targets(np.linspace(0, 1, n), np.zeros(n), oc, np.zeros(n, np.int32))
    u = torch.full((2, n), 2.0, dtype=torch.float64, device="cuda")
    with pytest.raises(s2d.S2DError) as ei:
        s2d.stokes2d_slp_eval(mode, src, t, 1.0, -1, 1, 1.0, u[0], u[1],
                              ws=torch.empty(0, dtype=torch.uint8, device="cuda"))
    assert ei.value.code == s2d.S2D_EWORKSPACE
    torch.cuda.synchronize()
    assert torch.all(u == 2.0)
    s2d.stokes2d_slp_eval(mode, src, t, 1.0, -1, 1, 1.0, u[0], u[1])
    torch.cuda.synchronize()
    nan = torch.as_tensor(oc >= 0, device="cuda")
    assert torch.isnan(u[:, nan]).all() and torch.all(u[:, ~nan] == 0)


# FP32C sums over a tile's own neighbourhood add float terms in FP64: the error
# is that of the terms' own roundings, emulated here (the hardware's reciprocal
# and logarithm may be off by one unit of the last place where the emulation
# has half of one, hence the factor; float sums of neighbouring terms or images
# double the error and more).
@pytest.mark.parametrize("img,d", [((0, 0), 1.0), ((-1, 1), 0.66)])
def test_float_terms_near_own_curves_are_added_in_fp64(img, d):
    import torch
    import paper_1510_05616_amd as s2d
    f32 = np.float32
    got, want = [], []
    for seed in range(12):
        rng = np.random.default_rng(seed)
        parts = []
        for i in range(2):
            t = 2 * np.pi * np.arange(64) / 64
            f = [sum((rng.normal() * np.cos(k * t) + rng.normal() * np.sin(k * t)) / k ** 2 for k in range(1, 7))
                 for _ in range(2)]
            c = synth.ellipse_curve(0.25, 0.14, 64, (0.13 * i, 0.68 * i), phi=rng.uniform(1, 2))
            parts.append((c.x, c.y, c.nx, c.ny, c.w, c.kappa, f[0], f[1]))
        cs = synth.concat_curves(parts)
        cur = np.repeat(np.arange(2, dtype=np.int32), 64)
        src, trg = s2d.Curves(cs), s2d.Targets(cs.x, cs.y, cur, np.arange(128, dtype=np.int32))
        r = []
        for mode in MODES:
            u = torch.zeros(2, 128, dtype=torch.float64, device="cuda")
            s2d.stokes2d_slp_eval(mode, src, trg, d, img[0], img[1], 1.0, u[0], u[1])
            r.append(u.cpu().numpy())
        got.append(r[1] - r[0])
        e = np.zeros((2, 128))
        gx, gy = cs.w * cs.fx, cs.w * cs.fy
        for n in range(img[0], img[1] + 1):
            rx, ry = cs.x[:, None] - n * d - cs.x[None], cs.y[:, None] - cs.y[None]
            on = (cur[:, None] != cur[None]) | (n != 0)
            q = np.where(on, rx * rx + ry * ry, 1.0)
            a, b, hx, hy = rx.astype(f32), ry.astype(f32), gx.astype(f32), gy.astype(f32)
            p = np.where(on, (a.astype(float) ** 2 + (b * b).astype(float)).astype(f32), f32(1))
            t = ((a.astype(float) * hx + (b * hy).astype(float)).astype(f32) * (f32(1) / p)).astype(f32)
            m, ex = np.frexp(p)
            l = -0.5 * np.log(2.0) * (ex + np.log2(m.astype(float)).astype(f32).astype(float))
            L, T = -0.5 * np.log(q), (rx * gx + ry * gy) / q
            e[0] += np.where(on, l * hx + (a * t).astype(float) - L * gx - rx * T, 0.0).sum(1)
            e[1] += np.where(on, l * hy + (b * t).astype(float) - L * gy - ry * T, 0.0).sum(1)
        want.append(e / (4 * np.pi))
    g, w = np.sqrt(np.mean(np.square(got))), np.sqrt(np.mean(np.square(want)))
    print(f"images {img}: FP32C error {g:.2e}, of the terms {w:.2e}", flush=True)
    assert 0 < g < 1.4 * w


# Few targets against sources that more than 64 split groups share (one and
# three target tiles, the last ragged; superblocks of 16 and of 64)
@pytest.mark.parametrize("n_trg,nodes", [(1, 150016), (64, 262145), (150, 300000)])
@pytest.mark.parametrize("mode", MODES)
def test_few_targets_many_split_groups(n_trg, nodes, mode):
    import torch
    import oracle
    import paper_1510_05616_amd as s2d
    c = synth.ellipse_curve(1.0, 0.6, nodes, fx=np.cos, fy=lambda t: np.sin(2 * t) + 0.3)
    rng = np.random.default_rng(n_trg)
    x, y = rng.uniform(-2, 2, n_trg), rng.uniform(0.8, 2, n_trg)
    src, t = s2d.Curves(c), s2d.Targets(x, y)
    u = torch.zeros(4, n_trg, dtype=torch.float64, device="cuda")
    s2d.stokes2d_slp_eval(mode, src, t, 5.0, -1, 1, 0.8, u[0], u[1])
    s2d.stokes2d_dlp_eval(mode, src, t, 5.0, -1, 1, u[2], u[3])
    torch.cuda.synchronize()
    g = u.cpu().numpy()
    o = *oracle.slp(c, x, y, d=5.0, img_lo=-1, img_hi=1, mu=0.8), *oracle.dlp(c, x, y, d=5.0, img_lo=-1, img_hi=1)
    for i in (0, 2):
        e = rel_err(g[i], g[i + 1], o[i], o[i + 1])
        print(f"{n_trg} targets, {nodes} sources, mode {mode}: {e:.2e}", flush=True)
        assert e <= TOL[mode]
