// Launch planning of one pair-sum evaluation: the launch shape (waves per
// workgroup, split groups per target tile) and the workspace carve-up.  Kept
// apart from the C ABI so that the pair kernels' sources and their planner
// can be fingerprinted together.
#include "s2d_internal.h"

#include <algorithm>
#include <cstdlib>

namespace s2d {

namespace {
size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
}  // namespace

size_t rec_bytes(int op, int mode) {
    if (slp_sources(op)) return mode == S2D_FP64 ? sizeof(RecSlp64) : sizeof(RecSlp32);
    return mode == S2D_FP64 ? sizeof(RecDlp64) : sizeof(RecDlp32);
}

Plan make_plan(int op, int mode, const s2d_curves *s, const s2d_targets *t, int cus) {
    Plan p{};
    p.op = op;
    p.mode = mode;
    p.tpt = 1;
    // Launch shape: one target tile (64 targets) per workgroup of W waves,
    // each wave a source split, and G split groups (workgroups) per tile.
    // G = 1 when the source records fit comfortably in one XCD's L2 (4 MB)
    // and the tiles alone give at least two rounds of 8 waves per SIMD;
    // otherwise G grows to fill the chip (few targets, many sources), and is
    // a multiple of 8 when the records exceed the L2 budget, so that every
    // XCD streams only its own groups' sources.  S2D_WAVES and S2D_GROUPS
    // override the shape for tuning sweeps.
    static const int env_waves = [] {
        const char *e = std::getenv("S2D_WAVES");
        const int v = e ? std::atoi(e) : 0;
        return (v >= 1 && v <= kMaxPairWaves) ? v : 0;
    }();
    static const int env_groups = [] {
        const char *e = std::getenv("S2D_GROUPS");
        return e ? std::max(0, std::atoi(e)) : 0;
    }();
    constexpr size_t kL2Budget = (size_t)3 << 20;
    p.n_src = s->n_nodes;
    p.n_trg = t->n;
    p.n_tiles = (p.n_trg + kWave - 1) / kWave;
    // Superblocks of 256 sources give every wave its split when there are
    // enough of them to fill the chip; few targets or sources leave waves idle
    // then, and a split of 64 or 16 sources is shorter (576 targets and 512
    // wall nodes: 2 waves of 256 sources a tile 126 us, 16 waves of 32 sources
    // 22 us; 10,496 targets and 4,096 wall nodes 134 and 52 us).
    const int64_t busy = (int64_t)cus * 16;
    p.sbs = kSuperBlock;
    while (p.sbs > kSubBlock && p.n_tiles * ((p.n_src + p.sbs - 1) / p.sbs) < busy) p.sbs /= 4;
    p.n_sb = (p.n_src + p.sbs - 1) / p.sbs;
    if (p.n_sb > 0 && p.n_tiles > 0) {
        const bool fits = (size_t)p.n_sb * p.sbs * rec_bytes(op, mode) <= kL2Budget;
        const int64_t fill = (int64_t)cus * 4 * 16;
        // a group's waves keep at least 64 sources each, and of more than 64
        // groups there are no more than give each CU four workgroups (eight are
        // up to a tenth faster and their planes twice the memory)
        const int64_t gmax = std::min<int64_t>(std::max<int64_t>(1, p.n_src / (64 * kMaxPairWaves)),
                                               std::max<int64_t>(64, (4 * (int64_t)cus + p.n_tiles - 1) / p.n_tiles));
        const bool by8 = !fits && gmax >= 8 && cus >= 8;
        int64_t G = 1;
        if (!(fits && p.n_tiles * kMaxPairWaves >= fill))
            G = std::min<int64_t>(std::max<int64_t>(1, (fill + p.n_tiles * kMaxPairWaves - 1) /
                                                           (p.n_tiles * kMaxPairWaves)), gmax);
        // Few workgroups: the group count with the least expected time.  A wave's
        // superblock of 256 sources takes a time unit (FP64 with three images
        // 121 us) with 16 waves on its CU, 1.8 with 32 and about 0.6 with 8; a
        // CU has as many workgroups as the fullest one of its XCD (groups go
        // round the XCDs where G is a multiple of 8), groups past the last source
        // are empty, and a plane costs about 1/500 unit.  1e6 sources, at most 64
        // groups: 64 targets 495 us, 640 targets 1.68 ms; by this rule 207 us and
        // 1.25 ms.
        if (G > 1 && p.n_tiles * std::min<int64_t>(G, 64) < 4 * (int64_t)cus) {
            const auto cost = [&](int64_t g) {
                const int64_t w = std::min<int64_t>(kMaxPairWaves, (p.n_sb + g - 1) / g);
                const int64_t sps = (p.n_sb + w * g - 1) / (w * g);
                const int64_t full = ((p.n_sb + sps - 1) / sps + w - 1) / w;         // groups that have sources
                const int64_t k = by8 ? (p.n_tiles * ((full + 7) / 8) + cus / 8 - 1) / (cus / 8)
                                      : (p.n_tiles * full + cus - 1) / cus;
                const double v = (double)(k * w) / kMaxPairWaves;
                return (double)(sps * p.sbs) / kSuperBlock * (v <= 1.0 ? 0.25 + 0.75 * v : 0.87 * v + 0.13) +
                       0.002 * (double)g;
            };
            const int64_t step = by8 ? 8 : 1;
            int64_t best = by8 ? 8 : 2;
            for (int64_t g = best; g <= gmax; g += step) best = cost(g) < cost(best) ? g : best;
            G = best;
        }
        if (by8) G = std::min<int64_t>((std::max<int64_t>(G, 8) + 7) / 8 * 8, gmax / 8 * 8);
        G = std::min<int64_t>(G, 65536);
        if (env_groups) G = std::min<int64_t>(env_groups, p.n_sb);
        // W: the full width, or fewer when the group has fewer superblocks.
        int W = (int)std::min<int64_t>(kMaxPairWaves, (p.n_sb + G - 1) / G);
        // Kress's rule is shared by all of a tile's waves, those without sources too
        if (op == S2D_OP_SLP && t->on_curve && G == 1) W = std::max(W, 16);
        if (env_waves) W = env_waves;
        p.waves = W;
        p.n_groups = (int)G;
        p.n_splits = (int)(W * G);
        p.sb_per_split = (p.n_sb + p.n_splits - 1) / p.n_splits;
        p.n_blocks = p.n_tiles * G;
    } else {
        p.waves = 1;
        p.n_groups = 1;
        p.sb_per_split = 0;
        p.n_splits = 0;
        p.n_blocks = 0;
    }
    p.self = false;    // set by the caller once images are known
    size_t off = 0;
    p.off_rec = off;
    off = align256(off + (size_t)p.n_sb * p.sbs * rec_bytes(op, mode));
    p.off_rec64 = off;
    if (mode == S2D_FP32C && s2d::near_fp64(op))
        off = align256(off + (size_t)p.n_sb * p.sbs * rec_bytes(op, S2D_FP64));
    p.off_sub = off;
    if (mode == S2D_FP32C)
        off = align256(off + (size_t)p.n_sb * (p.sbs / kSubBlock) * sizeof(s2d::SubInfo));
    p.off_sbsum = off;
    if (op == S2D_OP_SLP && mode == S2D_FP32C) off = align256(off + (size_t)p.n_sb * 2 * sizeof(double));
    // Kress's rule reads the sources while other tiles finish: outputs that lie
    // over them wait in a plane (api.hip)
    const bool own = op == S2D_OP_SLP && t->on_curve;
    p.off_part = off;
    if (p.n_groups > 1 || own) off = align256(off + (size_t)p.n_groups * 2 * (size_t)p.n_trg * sizeof(double));
    p.off_kress = off;
    if (own && p.n_trg > 0) off = align256(off + (size_t)p.n_src * sizeof(double));
    p.total = off;
    return p;
}

}  // namespace s2d
