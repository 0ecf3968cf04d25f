// Far-field summation of the layers' velocities, pressures and traction in FP64.
//
// A direct sum over the 128k channel's 2.8e10 (target, source, image) triples
// is bound by FP64 issue (15 ms) although all but about 1 % of the triples are
// far apart.  Here sources and targets are sorted along a Hilbert curve and
// cut into tiles of 64; a tile pair that is well separated interacts through
// expansions, the others term by term.
//
// Representation.  With complex z = x + i y and r = z - w both layers have the
// Goursat form
//   u = phi(z) - (z - c) conj(phi'(z)) + conj(psi(z)) + const
// (c any centre; psi depends on it):
//   single layer (g = w f):   phi = -1/2 sum g log r,
//     psi = -1/2 sum conj(g) log r - 1/2 sum conj(w - c) g / r,  const = 1/2 sum g
//   double layer (a = nu tau, b = 2 Re(conj(nu) tau)):  phi = 1/4 sum a / r,
//     psi = 1/4 [ sum b / r - sum conj(w - c) a / r^2 ],         const = 0
// and the other operators follow from the same two functions:
//   single-layer pressure sum Re(g / r) = -2 Re phi',
//   double-layer pressure sum Re(a / r^2) = -4 Re phi',
//   traction (normal m) -m Re phi' + 1/2 conj(m) conj(conj(z - c) phi'' - psi').
// So a cluster is two complex series of kOrder terms.  About a source centre
//   phi = a_0 log z + sum_{k>=1} a_k z^-k,  psi likewise (b_0 = conj(a_0));
// about a target centre at t = c_t - c_s, z = t + x,
//   alpha_l = (-1)^l t^-l [ sum_k C(l+k-1, l) a_k t^-k - a_0 / l ]
//   (alpha_0 with a_0 (log |t| - 1), the -1 being the constant),
//   beta_l the same of b_k, less conj(t) (l + 1) alpha_{l+1}.
// Only real parts of logarithms enter u: the arguments cancel between phi and
// conj(psi).
//
// Acceptance.  A source node of radius r_s and a target tile of radius r_t at
// distance D are far when r_s < th (D - r_t) and r_t < th (D - r_s), th = 0.32:
// the series' first dropped powers are 0.32^31 = 5e-16 (0.32^32 for a source
// node's), times the factors k that psi's and the derivatives' terms carry and a
// geometric tail of 1.5: an estimate of about 1e-15 of the terms' magnitudes in
// the worst place, not a bound.  Against the direct sums, with the density on one node, errors
// over |term| stay at rounding (largest 4.0e-15 for velocities, 6.1e-15 for
// pressures and traction) for th = 0.28 and 0.32 alike, double at 0.34 and are
// 2e-13 at 0.37; the channel step below takes 0.93, 0.87, 0.84 and 0.81 ms.
// Non-finite boxes never pass and are summed term by term.
// Source nodes have three levels (64, 1,024 and 16,384 sources); a target tile
// walks them from the top.  Coordinates inside the expansions are scaled by a
// power of two to about the domain's extent, and nodes closer than 1e-8 of it
// or 1e8 times its size are never far, so no power over- or underflows
// harmfully.  The domain is where the points are but for a few (far_keys):
// those far outside cost their own tiles term by term and nothing else.
//
// Measured (MI355X): single layer of 1,000 vesicles x 96 nodes at their own
// nodes (the channel's three rows, 64 pi long), images -1..1: 15.1 ms direct;
// here 0.23 ms near part, 0.17 ms far part, 0.06 ms own curves and source
// expansions, 0.1 ms set-up (once per geometry).  Walls of 2 x 16,000 nodes
// refined 8 times at 20,000 near-wall points: 8.6 ms direct; near and far parts
// of both sums 0.33 ms, set-up 0.1 ms each.  Both parts are bound by FP64 issue and the latency of its
// dependent chains at 3-5 waves per SIMD.
//
// Every sum runs in a fixed order (stable sort, ballots, no floating-point
// atomics): results repeat bit for bit.
#include "s2d_far.h"
#include "self_impl.h"

#include <algorithm>

namespace s2d {

namespace {

constexpr int kTile = 64;        // sources and targets per tile: one wave
constexpr int kFan = 16;         // children of a top node
constexpr int kLeafFan = 32;     // and of a middle one: 16 tiles of two circles
constexpr int kOrder = 32;       // coefficients per series, the logarithm's included
constexpr double kTheta = 0.32;
constexpr int kFarWaves = 4;     // waves per target tile, far kernel
constexpr int kNearWaves = 4;    // and near kernel
constexpr int kBoxBlocks = 64;
constexpr int kSortItems = 1024; // items per sort block
// bits of a sort key (the bit above marks targets), eight to a pass: cells of
// a few points at most where the points fill their domain evenly
constexpr int key_bits(int64_t n) { return n <= 1 << 15 ? 15 : n <= 1 << 20 ? 23 : 31; }

// circle around points [lo, hi) of a tile (empty: lo == hi); upper levels keep lo = 0, hi = 1
struct FarNode {
    double x, y, r;
    int32_t lo, hi;
};
// expansion scale 2^-e, its log, least distance of a far node and greatest
// radius of a far one or of its target
struct FarBox { double s, logs, dmin, rmax; };

// C(l + k - 1, l), l = 0..31, k = 1..31 (column 0 unused)
struct Binom { double v[kOrder][kOrder]; };
constexpr Binom make_binom() {
    Binom b{};
    for (int k = 1; k < kOrder; ++k) b.v[0][k] = 1.0;
    for (int l = 1; l < kOrder; ++l)
        for (int k = 1; k < kOrder; ++k) b.v[l][k] = b.v[l - 1][k] + b.v[l][k - 1];
    return b;
}
__device__ const Binom kBinom = make_binom();

struct C2 { double x, y; };
__device__ __forceinline__ C2 cmul(C2 a, C2 b) {
    return {__builtin_fma(a.x, b.x, -a.y * b.y), __builtin_fma(a.x, b.y, a.y * b.x)};
}
// orders a wave's LDS writes before its own later reads
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    __builtin_amdgcn_wave_barrier();
}

// z^n, 0 <= n < 32
__device__ __forceinline__ C2 cpow5(C2 z, int n) {
    C2 r{1.0, 0.0};
#pragma unroll
    for (int b = 0; b < 5; ++b) {
        const C2 p = cmul(r, z);
        const bool on = (n >> b) & 1;
        r.x = on ? p.x : r.x;
        r.y = on ? p.y : r.y;
        if (b < 4) z = C2{__builtin_fma(z.x, z.x, -z.y * z.y), 2.0 * z.x * z.y};
    }
    return r;
}

__device__ __forceinline__ double wmin(double v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v = fmin(v, __shfl_xor(v, m, kWave));
    return v;
}
__device__ __forceinline__ double wmax(double v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v = fmax(v, __shfl_xor(v, m, kWave));
    return v;
}

// ---------------------------------------------------------------------------
// set-up: bounding box, Hilbert keys, stable radix sort, tiles
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void far_box(int64_t ns, int64_t nt, const double *sx, const double *sy,
                                               const double *tx, const double *ty, double *box) {
    __shared__ double red[4][4];
    const double inf = __builtin_inf();
    double v[4] = {inf, -inf, inf, -inf};
    // 32 points at a time in turn: any 256 neighbours meet eight blocks in a row
    constexpr int kRun = 32;
    const int64_t first = (int64_t)(threadIdx.x / kRun) * (kRun * kBoxBlocks) + blockIdx.x * kRun + threadIdx.x % kRun;
#pragma unroll 4
    for (int64_t i = first; i < ns + nt; i += 256 * kBoxBlocks) {
        double x = i < ns ? sx[i] : tx[i - ns], y = i < ns ? sy[i] : ty[i - ns];
        x = fabs(x) < inf ? x : __builtin_nan("");      // which neither fmin nor fmax takes
        y = fabs(y) < inf ? y : __builtin_nan("");
        v[0] = fmin(v[0], x);
        v[1] = fmax(v[1], x);
        v[2] = fmin(v[2], y);
        v[3] = fmax(v[3], y);
    }
    const int w = threadIdx.x / kWave;
    for (int k = 0; k < 4; ++k) {
        const double r = (k & 1) ? wmax(v[k]) : wmin(v[k]);
        if ((threadIdx.x & 63) == 0) red[w][k] = r;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        double r = red[0][threadIdx.x];
        for (int q = 1; q < 4; ++q) r = (threadIdx.x & 1) ? fmax(r, red[q][threadIdx.x]) : fmin(r, red[q][threadIdx.x]);
        box[4 * blockIdx.x + threadIdx.x] = r;
    }
}

// index of cell (x, y) along the Hilbert curve of 2^bits x 2^bits cells
__device__ __forceinline__ uint32_t hilbert(uint32_t x, uint32_t y, int bits) {
    uint32_t d = 0;
    for (int b = bits - 1; b >= 0; --b) {
        const uint32_t rx = (x >> b) & 1, ry = (y >> b) & 1;
        d = (d << 2) | ((3 * rx) ^ ry);
        if (ry == 0) {
            const uint32_t m = (1u << b) - 1;
            uint32_t a = x & m, c = y & m;
            if (rx) {
                a = m - a;
                c = m - c;
            }
            x = c;
            y = a;
        }
    }
    return d;
}

// one coordinate over far_box's blocks (lo > hi: a block without points): the
// points' interval, and the one that each of the eight sets of blocks reaches
struct Span { double lo, hi, core0, core1; };
__device__ __forceinline__ Span box_span(double lo, double hi) {
    const double inf = __builtin_inf();
    if (!(lo <= hi)) {
        lo = inf;
        hi = -inf;
    }
#pragma unroll
    for (int m = 32; m >= 8; m >>= 1) {
        lo = fmin(lo, __shfl_xor(lo, m, kWave));
        hi = fmax(hi, __shfl_xor(hi, m, kWave));
    }
    // the eight sets' intervals, in each of their lanes
    Span s{lo, hi, lo, hi};
    if (!(lo <= hi)) {                              // a set without points says nothing
        s.core0 = -inf;
        s.core1 = inf;
    }
#pragma unroll
    for (int m = 4; m >= 1; m >>= 1) {
        s.lo = fmin(s.lo, __shfl_xor(s.lo, m, kWave));
        s.hi = fmax(s.hi, __shfl_xor(s.hi, m, kWave));
        s.core0 = fmax(s.core0, __shfl_xor(s.core0, m, kWave));
        s.core1 = fmin(s.core1, __shfl_xor(s.core1, m, kWave));
    }
    if (s.core0 > s.core1) {
        const double t = s.core0;
        s.core0 = s.core1;
        s.core1 = t;
    }
    return s;
}

// [0, inf] to [0, h], in order
__device__ __forceinline__ double drawn_in(double t, double h) { return h > 0.0 ? h * (1.0 - h / (h + t)) : 0.0; }

// Sort keys: the domain's longer side is cut into squares of the shorter
// side's length (at most 2^10 of them) and each square is filled by a Hilbert
// curve, which ends where the next square's begins; a single Hilbert curve
// over the bounding square of a long channel leaves the channel and returns
// elsewhere, and tiles across such a jump are ten times larger.
//
// The domain is the points' box.  Where that reaches beyond the core (what each
// of eight sets of points reaches: far_box's blocks by their number mod 8; a few
// hundred points next to one another, or some dozens anywhere, reach all of
// them) by more than the core's extent, the points outside the core are drawn
// in, in their order, to half its extent, and sorted before (west, south) and
// behind all others, so that a tile of both kinds is cut between them.  One of 28,800 targets at 1e30 channel
// lengths put all others into one cell: 2.96 ms instead of 0.19 for the single
// layer of as many sources.
__global__ __launch_bounds__(256) void far_keys(int64_t ns, int64_t nt, const double *sx, const double *sy,
                                                const double *tx, const double *ty, const double *box, int bits, FarBox *info,
                                                uint32_t *key, int32_t *idx) {
    const int lane = threadIdx.x & 63;
    const Span xs = box_span(box[4 * lane], box[4 * lane + 1]), ys = box_span(box[4 * lane + 2], box[4 * lane + 3]);
    const double reach = fmax(xs.core1 - xs.core0, ys.core1 - ys.core0);
    const bool west = xs.lo < xs.core0 - reach, east = xs.hi > xs.core1 + reach;
    const bool south = ys.lo < ys.core0 - reach, north = ys.hi > ys.core1 + reach;
    const double half = 0.5 * reach;
    const double x0 = west ? xs.core0 - half : xs.lo, x1 = east ? xs.core1 + half : xs.hi;
    const double y0 = south ? ys.core0 - half : ys.lo, y1 = north ? ys.core1 + half : ys.hi;
    const bool tall = y1 - y0 > x1 - x0;
    const double ext = fmax(x1 - x0, y1 - y0), wid = fmin(x1 - x0, y1 - y0);
    const bool ok = ext > 0.0 && ext < 1e300;
    const double side = fmax(wid, ext * (1.0 / 1024.0)) * (1.0 + 1e-9);
    const int nb = ok ? min(1024, (int)(ext / side) + 1) : 1;
    const bool outside = west || east || south || north;      // a strip before and one behind for those points
    const int strips = outside ? nb + 2 : nb;
    const int cells = (bits - (strips > 1 ? 32 - __builtin_clz((unsigned)(strips - 1)) : 0)) / 2;   // bits per coordinate
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i == 0) {
        const int e = ok ? __builtin_amdgcn_frexp_exp(ext) : 0;
        *info = FarBox{ldexp(1.0, -e), -(double)e * 6.93147180559945286227e-01, ok ? 1e-8 * ext : 1e300,
                       ok ? 1e8 * ext : 0.0};
    }
    if (i >= ns + nt) return;
    const bool t = i >= ns;
    double u = t ? tx[i - ns] : sx[i], v = t ? ty[i - ns] : sy[i];
    const bool w = west && u < xs.core0, e = east && u > xs.core1, s = south && v < ys.core0, n = north && v > ys.core1;
    if (w) u = xs.core0 - drawn_in(xs.core0 - u, half);
    if (e) u = xs.core1 + drawn_in(u - xs.core1, half);
    if (s) v = ys.core0 - drawn_in(ys.core0 - v, half);
    if (n) v = ys.core1 + drawn_in(v - ys.core1, half);
    u -= x0;
    v -= y0;
    if (tall) {
        const double c = u;
        u = v;
        v = c;
    }
    // NaN coordinates land in cell 0, infinite ones in an outermost cell
    const double is = ok ? 1.0 / side : 0.0, m = (double)((1 << cells) - 1), c = (double)(1 << cells);
    u = fmin(fmax(u * is, 0.0), (double)nb);
    const bool out = w || e || s || n;
    if (out) u /= (double)nb;
    const int b = out ? 0 : min((int)u, nb - 1);
    const int strip = !outside ? b : !out ? b + 1 : w || s ? 0 : nb + 1;
    const uint32_t cx = (uint32_t)fmin((u - (double)b) * c, m), cy = (uint32_t)fmin(fmax(v * is, 0.0) * c, m);
    key[i] = (uint32_t)strip << (2 * cells) | hilbert(cx, cy, cells) | (t ? 1u << bits : 0u);
    idx[i] = (int32_t)(t ? i - ns : i);
}

// inclusive prefix sum over the wave
__device__ __forceinline__ uint32_t wave_scan(uint32_t v, int lane) {
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) {
        const uint32_t o = __shfl_up(v, m, kWave);
        if (lane >= m) v += o;
    }
    return v;
}

// one pass of the radix sort over 8 key bits: per-block digit counts ...
__global__ __launch_bounds__(256) void far_hist(int64_t n, int64_t nblk, int shift, const uint32_t *key,
                                                uint32_t *hist) {
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t b0 = (int64_t)blockIdx.x * kSortItems;
    uint32_t k[kSortItems / 256];
#pragma unroll
    for (int r = 0; r < kSortItems / 256; ++r) {
        const int64_t i = b0 + r * 256 + threadIdx.x;
        k[r] = i < n ? key[i] : 0;
    }
#pragma unroll
    for (int r = 0; r < kSortItems / 256; ++r)
        if (b0 + r * 256 + threadIdx.x < n) atomicAdd(&h[(k[r] >> shift) & 255], 1u);
    __syncthreads();
    hist[(int64_t)threadIdx.x * nblk + blockIdx.x] = h[threadIdx.x];
}

// ... their exclusive prefix over the blocks of each digit (one wave each) ...
__global__ __launch_bounds__(256) void far_scan(int64_t nblk, uint32_t *hist, uint32_t *total) {
    const int lane = threadIdx.x & 63, dgt = blockIdx.x * 4 + threadIdx.x / 64;
    uint32_t *row = hist + (int64_t)dgt * nblk;
    uint32_t run = 0;
    for (int64_t b = 0; b < nblk; b += 64) {
        const uint32_t v = b + lane < nblk ? row[b + lane] : 0;
        const uint32_t s = wave_scan(v, lane);
        if (b + lane < nblk) row[b + lane] = run + s - v;
        run += __shfl(s, 63, kWave);
    }
    if (lane == 0) total[dgt] = run;
}

// ... and the scatter, in input order within a digit (stable).  Rounds of 256
// items, serial through the digits' running positions: a block's items are
// loaded before the first (a load in each round: 10.7 us a pass on 224,000
// items in blocks of 2,048, 7.9 with the loads ahead, 5.7 in blocks of 1,024;
// 512 gain nothing more and lengthen the scan).
__global__ __launch_bounds__(256) void far_scatter(int64_t n, int64_t nblk, int shift, const uint32_t *key,
                                                   const int32_t *idx, const uint32_t *hist, const uint32_t *total,
                                                   uint32_t *okey, int32_t *oidx) {
    __shared__ uint32_t run[256], cnt[4][256], wsum[4];
    const int lane = threadIdx.x & 63, wid = threadIdx.x / 64;
    // all of the block's items before its serial rounds
    const int64_t b0 = (int64_t)blockIdx.x * kSortItems;
    uint32_t keys[kSortItems / 256];
    int32_t ids[kSortItems / 256];
#pragma unroll
    for (int r = 0; r < kSortItems / 256; ++r) {
        const int64_t i = b0 + r * 256 + threadIdx.x;
        keys[r] = i < n ? key[i] : 0;
        ids[r] = i < n ? idx[i] : 0;
    }
    // the digits' first positions: an exclusive prefix of their totals
    const uint32_t v = total[threadIdx.x], s = wave_scan(v, lane);
    if (lane == 63) wsum[wid] = s;
    __syncthreads();
    uint32_t first = s - v;
    for (int q = 0; q < wid; ++q) first += wsum[q];
    run[threadIdx.x] = first + hist[(int64_t)threadIdx.x * nblk + blockIdx.x];
#pragma unroll
    for (int r = 0; r < kSortItems / 256; ++r) {
        for (int q = 0; q < 4; ++q) cnt[q][threadIdx.x] = 0;
        __syncthreads();
        const bool ok = b0 + r * 256 + threadIdx.x < n;
        const uint32_t k = keys[r];
        const int dgt = (k >> shift) & 255;
        uint64_t same = __ballot(ok);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const uint64_t m = __ballot((dgt >> b) & 1);
            same &= ((dgt >> b) & 1) ? m : ~m;
        }
        const int rank = __popcll(same & ((1ull << lane) - 1));
        if (ok && rank == 0) cnt[wid][dgt] = (uint32_t)__popcll(same);
        __syncthreads();
        if (ok) {
            uint32_t p = run[dgt] + rank;
            for (int q = 0; q < wid; ++q) p += cnt[q][dgt];
            okey[p] = k;
            oidx[p] = ids[r];
        }
        __syncthreads();
        run[threadIdx.x] += cnt[0][threadIdx.x] + cnt[1][threadIdx.x] + cnt[2][threadIdx.x] + cnt[3][threadIdx.x];
        __syncthreads();
    }
}

__device__ __forceinline__ FarNode far_circle(double x, double y, bool in, int lo, int hi) {
    const double inf = __builtin_inf();
    const double x0 = wmin(in ? x : inf), x1 = wmax(in ? x : -inf), y0 = wmin(in ? y : inf), y1 = wmax(in ? y : -inf);
    const double cx = 0.5 * (x0 + x1), cy = 0.5 * (y0 + y1), dx = x - cx, dy = y - cy;
    return FarNode{cx, cy, wmax(in ? sqrt(dx * dx + dy * dy) : 0.0) * (1.0 + 1e-12), lo, hi};
}

// Circles of the source and target tiles, the targets' sorted coordinates and
// the sources' sorted positions; one wave per tile.  A tile across a gap of the
// sort order (from one wall to the other, say) is cut at its widest gap into
// two circles where that halves its radius.
__global__ __launch_bounds__(256) void far_tiles(int64_t ns, int64_t nt, int64_t n0, int64_t nT, const double *sx,
                                                 const double *sy, const double *tx, const double *ty,
                                                 const int32_t *idx, int32_t *spos, FarNode *node, FarNode *tnode,
                                                 double *txy) {
    const int64_t t = (int64_t)blockIdx.x * 4 + threadIdx.x / 64;
    const int lane = threadIdx.x & 63;
    if (t >= n0 + nT) return;
    const bool src = t < n0;
    const int64_t p = (src ? t : t - n0) * kTile + lane, n = src ? ns : nt;
    const bool ok = p < n;
    const int count = (int)min((int64_t)kTile, n - (p - lane));
    double x = 0.0, y = 0.0;
    if (ok) {
        const int32_t o = idx[src ? p : ns + p];
        x = src ? sx[o] : tx[o];
        y = src ? sy[o] : ty[o];
        if (src) {
            spos[o] = (int32_t)p;
        } else {
            txy[p] = x;
            txy[nt + p] = y;
        }
        // a point that is not finite stays out of its circle, as a NaN does in
        // fmin and fmax: its own sum or its terms come out so in any case
        if (!(fabs(x) + fabs(y) < __builtin_inf())) x = y = __builtin_nan("");
    }
    const double gx = __shfl_down(x, 1, kWave) - x, gy = __shfl_down(y, 1, kWave) - y;
    const double gap = lane + 1 < count ? gx * gx + gy * gy : -1.0;
    const uint64_t at = __ballot(gap == wmax(gap) && gap > 0.0);
    FarNode a = far_circle(x, y, ok, 0, count), b{0.0, 0.0, 0.0, 0, 0};
    if (at) {                                        // wave-uniform
        const int cut = __builtin_ctzll(at) + 1;
        const FarNode l = far_circle(x, y, lane < cut, 0, cut), r = far_circle(x, y, lane >= cut && ok, cut, count);
        if (fmax(l.r, r.r) < 0.5 * a.r) {
            a = l;
            b = r;
        }
    }
    FarNode *o = src ? node + 2 * t : tnode + 2 * (t - n0);
    if (lane == 0) {
        o[0] = a;
        o[1] = b;
    }
}

// the circle around the children held by the lanes of a wave (`in`: this lane
// holds one)
__device__ __forceinline__ FarNode far_parent(const FarNode &c, bool in) {
    const double inf = __builtin_inf();
    const double x0 = wmin(in ? c.x - c.r : inf), x1 = wmax(in ? c.x + c.r : -inf);
    const double y0 = wmin(in ? c.y - c.r : inf), y1 = wmax(in ? c.y + c.r : -inf);
    const double cx = 0.5 * (x0 + x1), cy = 0.5 * (y0 + y1), dx = c.x - cx, dy = c.y - cy;
    return FarNode{cx, cy, wmax(in ? sqrt(dx * dx + dy * dy) + c.r : 0.0) * (1.0 + 1e-12), 0, 1};
}

// Circles of the upper levels: a workgroup per top node, a wave per middle
// node, a lane per leaf; n0: leaves (two per source tile).
__global__ __launch_bounds__(64 * kFan) void far_upper(int64_t n0, int64_t n1, FarNode *node) {
    __shared__ FarNode mid[kFan];
    const int wid = threadIdx.x / 64, lane = threadIdx.x & 63;
    const int64_t b = (int64_t)blockIdx.x * kFan, i = b + wid, c = i * kLeafFan + lane;
    if (i < n1) {
        FarNode l{0.0, 0.0, 0.0, 0, 0};
        if (lane < kLeafFan && c < n0) l = node[c];
        const FarNode p = far_parent(l, l.lo < l.hi);
        if (lane == 0) {
            mid[wid] = p;
            node[n0 + i] = p;
        }
    }
    __syncthreads();
    if (wid != 0) return;
    const bool in = lane < kFan && b + lane < n1;
    const FarNode p = far_parent(mid[in ? lane : 0], in);
    if (lane == 0) node[n0 + n1 + blockIdx.x] = p;
}

// ---------------------------------------------------------------------------
// source expansions
// ---------------------------------------------------------------------------
template <int OP>
using FRec = Rec64Of<OP>;

struct P2mArgs {
    int64_t ns, n0;
    const double *x, *y, *nx, *ny, *w, *fx, *fy;
    const int32_t *idx;
    const FarNode *node;
    const FarBox *info;
    void *rec;
    double *coef;              // per node [2 series][kOrder] complex
};

// Sorted records and the expansions of the leaves, one wave per leaf: each
// lane forms its source's terms four orders at a time, the wave's sum over
// the sources runs through LDS (16 rows, four lanes a row).
template <int OP>
__global__ __launch_bounds__(256) void far_p2m(P2mArgs a) {
    __shared__ double buf[4][16][kTile + 1];
    const int wid = threadIdx.x / 64, lane = threadIdx.x & 63;
    const int64_t t = (int64_t)blockIdx.x * 4 + wid;
    if (t >= a.n0) return;                          // no workgroup barrier below
    const FarNode nd = a.node[t];
    if (nd.lo == nd.hi) return;
    const int64_t p0 = (t >> 1) * kTile, p = p0 + lane;
    const bool ok = lane >= nd.lo && lane < nd.hi;
    const int32_t o = a.idx[ok ? p : p0 + nd.lo];
    const double X = a.x[o], Y = a.y[o], W = ok ? a.w[o] : 0.0;
    const double FX = ok ? a.fx[o] : 0.0, FY = ok ? a.fy[o] : 0.0;
    const double S = a.info->s;
    const C2 w{S * (X - nd.x), S * (Y - nd.y)};
    // lanes outside the leaf hold a copy of its first source with zero density
    C2 A, B;
    if (OP == S2D_OP_SLP) {
        if (ok) ((RecSlp64 *)a.rec)[p] = RecSlp64{X, Y, W * FX, W * FY};
        A = C2{0.5 * W * FX, 0.5 * W * FY};                        // g / 2
        B = C2{A.x, -A.y};
    } else {
        const double NX = ok ? W * a.nx[o] : 0.0, NY = ok ? W * a.ny[o] : 0.0;
        if (ok) ((RecDlp64 *)a.rec)[p] = RecDlp64{X, Y, NX, NY, FX, FY};
        A = C2{0.25 * S * (NX * FX - NY * FY), 0.25 * S * (NX * FY + NY * FX)};
        B = C2{0.5 * S * (NX * FX + NY * FY), 0.0};
    }
    const C2 wc{w.x, -w.y}, G = cmul(wc, A);         // conj(w) times the density
    C2 pw{1.0, 0.0}, pm{0.0, 0.0};                   // w^(k-1), w^(k-2)
#pragma unroll 1
    for (int k0 = 0; k0 < kOrder; k0 += 4) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = k0 + q;
            C2 ca, cb;
            if (k == 0) {
                const double z = OP == S2D_OP_SLP ? -1.0 : 0.0;
                ca = C2{z * A.x, z * A.y};
                cb = C2{z * B.x, z * B.y};
            } else {
                const C2 h = cmul(G, OP == S2D_OP_SLP ? pw : pm);
                const C2 nx = cmul(pw, w);           // w^k
                if (OP == S2D_OP_SLP) {
                    const double ik = 1.0 / (double)k;
                    const C2 u = cmul(A, nx), v = cmul(B, nx);
                    ca = C2{ik * u.x, ik * u.y};
                    cb = C2{__builtin_fma(ik, v.x, -h.x), __builtin_fma(ik, v.y, -h.y)};
                } else {
                    const double km = (double)(k - 1);
                    ca = cmul(A, pw);
                    cb = C2{__builtin_fma(-km, h.x, B.x * pw.x), __builtin_fma(-km, h.y, B.x * pw.y)};
                }
                pm = pw;
                pw = nx;
            }
            buf[wid][4 * q][lane] = ca.x;
            buf[wid][4 * q + 1][lane] = ca.y;
            buf[wid][4 * q + 2][lane] = cb.x;
            buf[wid][4 * q + 3][lane] = cb.y;
        }
        wave_lds_sync();
        const int row = lane >> 2, c0 = lane & 3;
        double s = 0.0;
#pragma unroll
        for (int j = 0; j < 16; ++j) s += buf[wid][row][4 * j + c0];
        s += __shfl_xor(s, 1, kWave);
        s += __shfl_xor(s, 2, kWave);
        wave_lds_sync();
        // row = 4 (order) + 2 (series) + part
        const int k = k0 + (row >> 2), h = (row >> 1) & 1;
        if (c0 == 0) a.coef[t * (4 * kOrder) + 2 * (h * kOrder + k) + (row & 1)] = s;
    }
}

// Expansions of an upper level: one workgroup per parent; a wave moves a
// child's series to the parent's centre, s = c_child - c_parent:
//   b_k += conj(s) phi'_k first (the change of psi's centre), then
//   new_k = sum_{j=1..k} C(k-1, j-1) s^(k-j) old_j - old_0 s^k / k
// (lane = series * kOrder + k); wave w takes children w, w + kFan, ... of
// `fan`, wave 0 adds the waves' sums in order.
__global__ __launch_bounds__(64 * kFan) void far_m2m(int64_t first, int64_t n_child, int fan, int64_t parent0,
                                                     const FarNode *node, const FarBox *info, double *coef) {
    __shared__ C2 old[kFan][2][kOrder], pw[kFan][kOrder + 1], sum[kFan][64];
    const int wid = threadIdx.x / 64, lane = threadIdx.x & 63, h = lane >> 5, k = lane & 31;
    const int64_t par = parent0 + blockIdx.x;
    const FarNode pn = node[par];
    C2 r{0.0, 0.0};
    for (int q0 = wid; q0 < fan; q0 += kFan) {
        const int64_t ci = (int64_t)blockIdx.x * fan + q0;
        if (ci >= n_child) break;
        const FarNode cn = node[first + ci];
        if (cn.lo == cn.hi) continue;
        const C2 s{info->s * (cn.x - pn.x), info->s * (cn.y - pn.y)};
        const C2 *cc = (const C2 *)coef + (first + ci) * 64;
        C2 m = cc[lane];
        if (h == 1 && k > 0) {
            C2 ph = cc[k - 1];
            if (k > 1) ph = C2{-(double)(k - 1) * ph.x, -(double)(k - 1) * ph.y};
            const C2 q = cmul(C2{s.x, -s.y}, ph);
            m.x += q.x;
            m.y += q.y;
        }
        old[wid][h][k] = m;
        const C2 sk = cpow5(s, k);
        if (h == 0) pw[wid][k] = sk;
        wave_lds_sync();
        if (k == 0) {
            r.x += m.x;
            r.y += m.y;
        } else {
            const C2 l = cmul(old[wid][h][0], sk);
            r.x -= l.x / (double)k;
            r.y -= l.y / (double)k;
            for (int j = 1; j <= k; ++j) {
                const C2 v = cmul(old[wid][h][j], pw[wid][k - j]);
                const double b = kBinom.v[j - 1][k - j + 1];
                r.x = __builtin_fma(b, v.x, r.x);
                r.y = __builtin_fma(b, v.y, r.y);
            }
        }
        wave_lds_sync();
    }
    sum[wid][lane] = r;
    __syncthreads();
    if (wid != 0) return;
    for (int q = 1; q < kFan; ++q) {
        r.x += sum[q][lane].x;
        r.y += sum[q][lane].y;
    }
    ((C2 *)coef)[par * 64 + lane] = r;
}

// ---------------------------------------------------------------------------
// the walk of one target tile over the source nodes and images
// ---------------------------------------------------------------------------
struct WalkArgs {
    int64_t n0, n1, n2;
    const FarNode *node;       // levels 0, 1, 2 one after another
    double d;
    int32_t img_lo, n_img;
};

// (a target circle without a finite centre is far from everything: its sums,
// term by term or not, are not numbers)
struct FarRange { double dmin, rmax; };
__device__ __forceinline__ bool far_from(const FarNode &t, const FarNode &s, double shift, const FarRange &in) {
    const double dx = t.x - (s.x + shift), dy = t.y - s.y;
    const double D = sqrt(__builtin_fma(dx, dx, dy * dy));
    if (!(fabs(t.x) + fabs(t.y) < __builtin_inf())) return true;
    return t.r < kTheta * (D - s.r) && s.r < kTheta * (D - t.r) && D > in.dmin && D < 1e300 &&
           fmax(t.r, s.r) < in.rmax;
}

// What a workgroup's waves share of a walk: the near top items of one chunk,
// their children's masks, the near middle nodes and their leaves' masks.
struct WalkLds {
    int top[kWave], mid[kWave * kFan], img[kWave * kFan];
    uint32_t far1[kWave], near1[kWave], far0[kWave * kFan], near0[kWave * kFan];
};

// Walks the source nodes and images for one target circle; called by all W
// waves of a workgroup.  The tests of the middle and lowest level are shared
// out and their masks meet in LDS (a wave walking alone spent as long on its
// tests as on its terms).  Then far(node, image) runs for the far nodes of
// every level (node: its place in `node`), or near(leaf, image) for the leaves
// summed term by term; the waves take them in turn in a fixed order, of which
// this one's are number `mine` of every `all`.
template <int W, bool FAR, class Fn>
__device__ __forceinline__ void far_walk(const WalkArgs &a, const FarNode &t, const FarRange &in, int wid, int lane, int mine,
                                         int all, WalkLds &sh, Fn &&fn) {
    const int n2 = (int)a.n2, items = n2 * a.n_img;
    int turn = 0;
    const auto take = [&](uint32_t mask, int64_t node0, int img) {
        for (; mask; mask &= mask - 1) {
            if (turn == mine) fn(node0 + __builtin_ctz(mask), img);
            turn = turn + 1 == all ? 0 : turn + 1;
        }
    };
    for (int b0 = 0; b0 < items; b0 += kWave) {
        const int it = b0 + lane;
        bool far = false;
        if (it < items) {
            const int q = it / n2;
            far = far_from(t, a.node[a.n0 + a.n1 + (it - q * n2)], (double)(a.img_lo + q) * a.d, in);
        }
        const uint64_t far2 = __ballot(far), near2 = __ballot(it < items && !far);
        const int nA = __popcll(near2);
        if (wid == 0 && it < items && !far) sh.top[__popcll(near2 & ((1ull << lane) - 1))] = it;
        __syncthreads();
        for (int q = wid; q < nA; q += W) {
            const int item = __builtin_amdgcn_readfirstlane(sh.top[q]), im = item / n2, i2 = item - im * n2;
            const int64_t c = (int64_t)i2 * kFan + lane;
            const bool ok = lane < kFan && c < a.n1;
            const bool f = ok && far_from(t, a.node[a.n0 + c], (double)(a.img_lo + im) * a.d, in);
            const uint64_t mf = __ballot(f), mn = __ballot(ok && !f);
            if (lane == 0) {
                sh.far1[q] = (uint32_t)mf;
                sh.near1[q] = (uint32_t)mn;
            }
        }
        __syncthreads();
        const uint32_t m1 = lane < nA ? sh.near1[lane] : 0;
        const int up = (int)wave_scan(__popc(m1), lane), nB = __builtin_amdgcn_readlane(up, kWave - 1);
        if (wid == 0 && lane < nA) {
            const int item = sh.top[lane], im = item / n2;
            int at = up - __popc(m1);
            for (uint32_t m = m1; m; m &= m - 1, ++at) {
                sh.mid[at] = (item - im * n2) * kFan + __builtin_ctz(m);
                sh.img[at] = a.img_lo + im;
            }
        }
        __syncthreads();
        for (int q = wid; q < nB; q += W) {
            const int i1 = __builtin_amdgcn_readfirstlane(sh.mid[q]), im = __builtin_amdgcn_readfirstlane(sh.img[q]);
            const int64_t c = (int64_t)i1 * kLeafFan + lane;
            bool ok = lane < kLeafFan && c < a.n0, f = false;
            if (ok) {
                const FarNode s = a.node[c];
                ok = s.lo < s.hi;
                f = ok && far_from(t, s, (double)im * a.d, in);
            }
            const uint64_t mf = __ballot(f), mn = __ballot(ok && !f);
            if (lane == 0) {
                sh.far0[q] = (uint32_t)mf;
                sh.near0[q] = (uint32_t)mn;
            }
        }
        __syncthreads();
        if (FAR) {
            for (uint64_t m = far2; m; m &= m - 1) {
                const int item = b0 + __builtin_ctzll(m), im = item / n2;
                take(1, a.n0 + a.n1 + (item - im * n2), a.img_lo + im);
            }
            for (int q = 0; q < nA; ++q) {
                const int item = __builtin_amdgcn_readfirstlane(sh.top[q]), im = item / n2;
                take(__builtin_amdgcn_readfirstlane(sh.far1[q]), a.n0 + (int64_t)(item - im * n2) * kFan,
                     a.img_lo + im);
            }
        }
        for (int q = 0; q < nB; ++q)
            take(__builtin_amdgcn_readfirstlane(FAR ? sh.far0[q] : sh.near0[q]),
                 (int64_t)__builtin_amdgcn_readfirstlane(sh.mid[q]) * kLeafFan,
                 __builtin_amdgcn_readfirstlane(sh.img[q]));
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// far part: the target tile's local expansion and its values
// ---------------------------------------------------------------------------
// The circle of workgroup `blk` of n (two per tile): all first circles, then
// the second ones, most of them empty; workgroups go round-robin to the XCDs,
// so taking them alternately would leave every second XCD idle.
__device__ __forceinline__ int far_circle_of(int blk, int n) { return blk < n / 2 ? 2 * blk : 2 * (blk - n / 2) + 1; }

struct FarArgs {
    WalkArgs w;
    int64_t nt;
    const FarNode *tnode;
    const FarBox *info;
    const double *coef, *txy;
    double *part;              // [2][nt], sorted targets
    const int32_t *tidx;
    const double *tnx, *tny;   // target normals (traction), caller's order
};

// One workgroup per target circle; its waves take the far nodes in turn.  Lane
// (series, l) holds local coefficient l and row l of the binomial table; the
// 2 x 31 scaled source coefficients pass through LDS.
template <int OP>
__global__ __launch_bounds__(64 * kFarWaves) __attribute__((amdgpu_waves_per_eu(4, 4)))
void far_far(FarArgs a) {
    __shared__ C2 buf[kFarWaves][2][kOrder + 1], sum[kFarWaves][2][64], la[kFarWaves][slp_sources(OP) ? kWave : 1];
    __shared__ double lq[kFarWaves][slp_sources(OP) ? kWave : 1];
    __shared__ WalkLds sh;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x & 63;
    const int h = lane >> 5, l = lane & 31;
    const int circle = far_circle_of(blockIdx.x, gridDim.x);
    const FarNode t = a.tnode[circle];
    if (t.lo == t.hi) return;
    const double S = a.info->s, logs = a.info->logs;
    double row[kOrder];
#pragma unroll
    for (int k = 1; k < kOrder; ++k) row[k] = kBinom.v[l][k];
    const double sgn = (l & 1) ? -1.0 : 1.0, il = l ? -1.0 / (double)l : h == 0 ? -1.0 : 0.0;
    C2 acc{0.0, 0.0}, gam{0.0, 0.0}, lsum{0.0, 0.0};
    // a_0 log |t| of the nodes held in LDS, summed over the lanes' own share
    int held = 0;
    const auto flush = [&] {
        if (lane < held) {
            const double c = __builtin_fma(0.5, log64(lq[wid][lane]), -logs);
            lsum.x = __builtin_fma(la[wid][lane].x, c, lsum.x);
            lsum.y = __builtin_fma(la[wid][lane].y, c, lsum.y);
        }
        held = 0;
    };
    far_walk<kFarWaves, true>(
        a.w, t, FarRange{a.info->dmin, a.info->rmax}, wid, lane, wid, kFarWaves, sh, [&](int64_t at, int img) {
            const FarNode s = load_ro<FarNode>(a.w.node, at);
            const C2 m = ((const C2 *)a.coef)[at * 64 + lane];
            const C2 tt{S * (t.x - (s.x + (double)img * a.w.d)), S * (t.y - s.y)};
            const double q = __builtin_fma(tt.x, tt.x, tt.y * tt.y), iq = rcp64(q);
            // terms until (r_s / (D - r_t))^k < 2^-56
            const float ratio = (float)(S * s.r) * __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf((float)q) - (float)(S * t.r));
            const int terms = __builtin_amdgcn_readfirstlane(
                min(kOrder - 1, max(1, (int)(-56.0f / __builtin_amdgcn_logf(ratio)) + 2)));
            const C2 e = cpow5(C2{tt.x * iq, -tt.y * iq}, l);        // t^-l
            buf[wid][h][l] = l ? cmul(m, e) : m;
            wave_lds_sync();
            C2 v{0.0, 0.0};
#pragma unroll
            for (int k0 = 1; k0 < kOrder; k0 += 4) {
                if (k0 > terms) break;
#pragma unroll
                for (int k = k0; k < k0 + 4 && k < kOrder; ++k) {
                    const C2 b = buf[wid][h][k];
                    v.x = __builtin_fma(row[k], b.x, v.x);
                    v.y = __builtin_fma(row[k], b.y, v.y);
                }
            }
            if (slp_sources(OP)) {
                const C2 m0 = buf[wid][h][0];
                v.x = __builtin_fma(m0.x, il, v.x);
                v.y = __builtin_fma(m0.y, il, v.y);
                // the logarithms of 64 nodes at a time, a lane each
                if (lane == 0) {
                    lq[wid][held] = q;
                    la[wid][held] = m0;
                }
                if (++held == kWave) {
                    wave_lds_sync();
                    flush();
                }
            }
            wave_lds_sync();
            C2 r = cmul(v, e);
            r.x *= sgn;
            r.y *= sgn;
            acc.x += r.x;
            acc.y += r.y;
            const C2 g = cmul(C2{tt.x, -tt.y}, r);
            gam.x += g.x;
            gam.y += g.y;
        });
    if (slp_sources(OP)) {
        wave_lds_sync();
        flush();
#pragma unroll
        for (int m = kWave / 2; m >= 1; m >>= 1) {
            lsum.x += __shfl_xor(lsum.x, m, kWave);
            lsum.y += __shfl_xor(lsum.y, m, kWave);
        }
        // phi_0 with a_0 log |t|, psi_0 with its conjugate
        if (l == 0) {
            acc.x += lsum.x;
            acc.y += h == 0 ? lsum.y : -lsum.y;
        }
    }
    sum[wid][0][lane] = acc;
    sum[wid][1][lane] = gam;
    __syncthreads();
    if (wid != 0) return;
    for (int w = 1; w < kFarWaves; ++w) {
        acc.x += sum[w][0][lane].x;
        acc.y += sum[w][0][lane].y;
        gam.x += sum[w][1][lane].x;
        gam.y += sum[w][1][lane].y;
    }
    sum[0][1][lane] = gam;
    wave_lds_sync();
    if (h == 1 && l + 1 < kOrder) {
        const C2 g = sum[0][1][l + 1];
        acc.x = __builtin_fma(-(double)(l + 1), g.x, acc.x);
        acc.y = __builtin_fma(-(double)(l + 1), g.y, acc.y);
    }
    sum[0][0][lane] = acc;
    wave_lds_sync();
    const int64_t p = (int64_t)(circle >> 1) * kTile + lane;
    if (lane < t.lo || lane >= t.hi) return;
    const C2 x{S * (a.txy[p] - t.x), S * (a.txy[a.nt + p] - t.y)};
    // phi, phi', phi'' / 2, psi, psi' by Horner's rule (unused ones drop out)
    C2 f{0.0, 0.0}, df{0.0, 0.0}, d2{0.0, 0.0}, g{0.0, 0.0}, dg{0.0, 0.0};
    const auto step = [&](C2 &v, C2 add) {
        const C2 c = cmul(v, x);
        v = C2{c.x + add.x, c.y + add.y};
    };
    for (int k = kOrder - 1; k >= 0; --k) {
        if (OP == S2D_OP_SLP_TRACTION) {
            step(d2, df);
            step(dg, g);
        }
        step(df, f);
        step(f, sum[0][0][k]);
        if (OP <= S2D_OP_DLP || OP == S2D_OP_SLP_TRACTION) step(g, sum[0][0][32 + k]);
    }
    double ox, oy = 0.0;
    if (OP <= S2D_OP_DLP) {
        // phi - x conj(phi') + conj(psi)
        ox = f.x - (x.x * df.x + x.y * df.y) + g.x;
        oy = f.y - (x.y * df.x - x.x * df.y) - g.y;
    } else if (OP == S2D_OP_SLP_TRACTION) {
        const int32_t i = a.tidx[p];
        const C2 m{a.tnx[i], a.tny[i]}, q = cmul(C2{x.x, -x.y}, d2);
        // conj(m (conj(x) phi'' - psi')) / 2
        const C2 v = cmul(m, C2{q.x - 0.5 * dg.x, q.y - 0.5 * dg.y});
        ox = S * (v.x - m.x * df.x);
        oy = S * (-v.y - m.y * df.x);
    } else {
        ox = (OP == S2D_OP_SLP_PRESSURE ? -2.0 : -4.0) * S * df.x;
    }
    a.part[p] = ox;
    a.part[a.nt + p] = oy;
}

// ---------------------------------------------------------------------------
// near part: the remaining tiles term by term, and the final step
// ---------------------------------------------------------------------------
struct NearArgs {
    WalkArgs w;
    int64_t ns, nt;
    int n_groups;
    const FarNode *tnode;
    const FarBox *info;
    const void *rec;
    const double *txy;
    double *part;                          // planes [2][nt]: the far part, then the groups' when n_groups > 1
    const int32_t *tidx, *spos;
    const int32_t *on_curve, *on_node;     // NULL when no target sits on a source node (or n = 0 is not summed)
    const double *tnx, *tny;               // target normals (traction)
};

// n_groups workgroups per target circle; their waves take the near leaves in
// turn, a record wave-uniform through the scalar path as in pair_sum().  A
// target's own source node is skipped at image 0; the own-curve terms of
// Kress's rule are added in final_one().
template <int OP>
__global__ __launch_bounds__(64 * kNearWaves) void far_near(NearArgs a, FinalArgs f) {
    __shared__ __attribute__((aligned(16))) double ltab[kLogTabWords];
    __shared__ double red[2][kNearWaves - 1][kWave];
    __shared__ WalkLds sh;
    const int blk = blockIdx.x / a.n_groups, group = blockIdx.x - blk * a.n_groups;
    const int circle = far_circle_of(blk, gridDim.x / a.n_groups);
    const FarNode t = a.tnode[circle];
    if (t.lo == t.hi) return;
    if (OP == S2D_OP_SLP) fill_log_table(ltab);
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x & 63;
    const int64_t p = (int64_t)(circle >> 1) * kTile + lane;
    const bool act = lane >= t.lo && lane < t.hi;
    const double tx = act ? a.txy[p] : t.x, ty = act ? a.txy[a.nt + p] : t.y;
    const int32_t i = act ? a.tidx[p] : 0;
    int self = -1;
    if (act && a.on_curve && a.on_curve[i] >= 0) {
        const int j = a.on_node[i];
        if (j >= 0 && j < a.ns) self = a.spos[j];
    }
    const bool tr = OP == S2D_OP_SLP_TRACTION && act;
    const double mx = tr ? a.tnx[i] : 0.0, my = tr ? a.tny[i] : 0.0;
    double ux = 0.0, uy = 0.0, lx = 0.0, ly = 0.0;
    far_walk<kNearWaves, false>(
        a.w, t, FarRange{a.info->dmin, a.info->rmax}, wid, lane, group * kNearWaves + wid, a.n_groups * kNearWaves, sh,
        [&](int64_t leaf, int img) {
            const double px[1] = {tx - (double)img * a.w.d};
            const int64_t at = (int64_t)(leaf >> 1) * kTile;
            const FRec<OP> *rec = (const FRec<OP> *)a.rec + at;
            const int u1 = load_ro<int32_t>(&a.w.node[leaf].hi, 0);
            int u = load_ro<int32_t>(&a.w.node[leaf].lo, 0);
            const int own = img == 0 && self >= 0 ? (int)(self - at) : -1;
            if (__ballot(own >= u && own < u1) == 0) {
                for (; u + 4 <= u1; u += 4) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const FRec<OP> s = load_ro<FRec<OP>>(rec, u + q);
                        if constexpr (OP == S2D_OP_SLP)
                            slp64_src<1>(px, ty, s, ltab, lx, ly, ux, uy);
                        else
                            rat64<OP>(px[0], ty, s, mx, my, ux, uy);
                    }
                }
            }
            for (; u < u1; ++u) {
                const FRec<OP> s = load_ro<FRec<OP>>(rec, u);
                double ax = 0.0, ay = 0.0, bx = 0.0, by = 0.0;
                if constexpr (OP == S2D_OP_SLP)
                    slp64_src<1>(px, ty, s, ltab, ax, ay, bx, by);
                else
                    rat64<OP>(px[0], ty, s, mx, my, bx, by);
                const bool ok = u != own;
                ux += ok ? bx : 0.0;
                uy += ok ? by : 0.0;
                if (OP == S2D_OP_SLP) {
                    lx += ok ? ax : 0.0;
                    ly += ok ? ay : 0.0;
                }
            }
        });
    if (OP == S2D_OP_SLP) {
        ux = __builtin_fma(-0.5, lx, ux);
        uy = __builtin_fma(-0.5, ly, uy);
    }
    if (wid > 0) {
        red[0][wid - 1][lane] = ux;
        red[1][wid - 1][lane] = uy;
    }
    __syncthreads();
    if (wid != 0 || !act) return;
    for (int w = 0; w < kNearWaves - 1; ++w) {
        ux += red[0][w][lane];
        uy += red[1][w][lane];
    }
    if (a.n_groups > 1) {
        double *o = a.part + (int64_t)(2 * (group + 1)) * a.nt;
        o[p] = ux;
        o[a.nt + p] = uy;
        return;
    }
    final_one(f, i, ux + a.part[p], uy + a.part[a.nt + p]);
}

// the far part and the groups' near parts, in order, and the final step
__global__ __launch_bounds__(256) void far_final(int64_t nt, int planes, const double *part, const int32_t *tidx,
                                                 FinalArgs f) {
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= nt) return;
    double sx = 0.0, sy = 0.0;
    for (int q = planes - 1; q >= 0; --q) {
        sx += part[(int64_t)(2 * q) * nt + p];
        sy += part[(int64_t)(2 * q + 1) * nt + p];
    }
    final_one(f, tidx[p], sx, sy);
}

// Kress's rule less the terms the sum above already holds (all own-curve
// nodes but the target's): sum_k T_(i-k) g_k, with the self node's
// [T_0 - log|x'|] g + t t^T g.
__global__ __launch_bounds__(256) void far_self(int64_t nt, int64_t ns, const int32_t *on_curve,
                                                const int32_t *on_node, const int32_t *off, int32_t nc,
                                                const double *nx, const double *ny, const double *w,
                                                const double *fx, const double *fy, const double *T, double *self) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= nt) return;
    const int c = on_curve[i];
    double sx = 0.0, sy = 0.0;
    if (c >= 0) {
        int lo = 0, N = 0, gi = -1;
        if (c < nc) {
            lo = off[c];
            N = off[c + 1] - lo;
            gi = on_node[i];
        }
        if (c >= nc || N < 2 || (N & 1) || lo < 0 || (int64_t)lo + N > ns || gi < lo || gi >= lo + N) {
            sx = sy = __builtin_nan("");
        } else {
            int m = gi - lo;
#pragma unroll 4
            for (int k = 0; k < N; ++k) {
                const double tw = T[lo + m] * w[lo + k];
                sx = __builtin_fma(tw, fx[lo + k], sx);
                sy = __builtin_fma(tw, fy[lo + k], sy);
                m = m == 0 ? N - 1 : m - 1;
            }
            const double gx = w[gi] * fx[gi], gy = w[gi] * fy[gi];
            const double ls = 1.0 - log(w[gi] * (double)N * 0.15915494309189535);   // N / (2 pi)
            const double ng = nx[gi] * gx + ny[gi] * gy;
            sx += ls * gx - nx[gi] * ng;
            sy += ls * gy - ny[gi] * ng;
        }
    }
    self[i] = sx;
    self[nt + i] = sy;
}

__global__ __launch_bounds__(256) void far_kress(const int32_t *off, int32_t nc, int64_t ns, double *T) {
    __shared__ double ctab[kCosTab];
    kress_table_curve(off, blockIdx.x, ns, T, ctab);
}

size_t al(size_t x) { return (x + 255) & ~(size_t)255; }

// the index array that holds the order after the last sort pass
size_t far_sorted(const FarLayout &L) { return L.idx[((L.bits + 1) / 8) & 1]; }

}  // namespace

FarLayout far_layout(int op, int64_t ns, int64_t nt, bool on_curve) {
    FarLayout L{};
    L.ns = ns;
    L.nt = nt;
    L.n0 = 2 * ((ns + kTile - 1) / kTile);
    L.n1 = (L.n0 + kLeafFan - 1) / kLeafFan;
    L.n2 = (L.n1 + kFan - 1) / kFan;
    L.nT = 2 * ((nt + kTile - 1) / kTile);
    // groups per circle: about eight near workgroups for each compute unit
    L.groups = (int)std::min<int64_t>(16, std::max<int64_t>(1, 4096 / std::max<int64_t>(L.nT, 1)));
    const size_t N = (size_t)(ns + nt);
    L.bits = key_bits((int64_t)N);
    L.nblk = (int64_t)((N + kSortItems - 1) / kSortItems);
    size_t o = 0;
    const auto take = [&](size_t bytes) {
        const size_t at = o;
        o = al(o + bytes);
        return at;
    };
    for (int k = 0; k < 2; ++k) {
        L.key[k] = take(N * sizeof(uint32_t));
        L.idx[k] = take(N * sizeof(int32_t));
    }
    L.hist = take((size_t)L.nblk * 256 * sizeof(uint32_t));
    L.base = take(256 * sizeof(uint32_t));
    L.box = take(4 * kBoxBlocks * sizeof(double) + sizeof(FarBox));
    L.spos = take((size_t)ns * sizeof(int32_t));
    L.node = take((size_t)(L.n0 + L.n1 + L.n2) * sizeof(FarNode));
    L.tnode = take((size_t)L.nT * sizeof(FarNode));
    L.txy = take(2 * (size_t)nt * sizeof(double));
    L.rec = take((size_t)ns * rec_bytes(op, S2D_FP64));
    L.coef = take((size_t)(L.n0 + L.n1 + L.n2) * 4 * kOrder * sizeof(double));
    // one plane and the groups' (groups * nt <= 131,072 by the rule above, so the size grows with nt)
    L.part = take(2 * ((size_t)nt + std::min<size_t>(16 * (size_t)nt, 131072)) * sizeof(double));
    L.kress = L.self = o;
    if (op == S2D_OP_SLP && on_curve) {
        L.kress = take((size_t)ns * sizeof(double));
        L.self = take(2 * (size_t)nt * sizeof(double));
    }
    L.total = o;
    return L;
}

// A direct sum takes about 22 us and kDirect[op][mode][images not grouped by
// three] us per 2^20 (source, target, image) triples; the far-field one, set-up
// included, about 140 us, 0.45 us per 1,000 sources, 1 us per 1,000 targets and
// 0.6 us for every source per target (a target tile's share of near sources
// grows as targets thin out), hardly more for three images than for one.  Far / direct, us, images -1..1,
// FP64 single layer, its pressure, FP32C single layer: 2,496 sources x 30,000
// targets 148 / 145, 130 / 90, 147 / 88; 9,984 x 14,000 151 / 270, 136 / 162, 150
// / 152; 60,000 x 5,000 181 / 646, 162 / 395, 182 / 365; 256,000 x 1,100 416 / 538,
// 385 / 327, 415 / 293; 256,000 x 3,000 274 / 1,502, 253 / 904, 275 / 796.  With a
// set-up for several densities (about 80 us) the velocities' lines lie at half
// the size.
bool far_worth(int op, int mode, int64_t ns, int64_t nt, int n_img, bool reuse) {
    static const double kDirect[5][2][2] = {{{0.66, 1.10}, {0.35, 0.56}},
                                            {{0.59, 0.74}, {0.37, 0.52}},
                                            {{0.40, 0.51}, {0.29, 0.41}},
                                            {{0.60, 0.83}, {0.38, 0.58}},
                                            {{0.60, 0.74}, {0.42, 0.49}}};
    if (op < S2D_OP_SLP || op > S2D_OP_SLP_TRACTION || ns < 2048 || nt < 1024 || ns + nt >= (int64_t)1 << 28) return false;
    const double triples = (double)ns * (double)nt * std::min(n_img, 3);
    if (reuse) return triples >= (double)(3 << 25);
    const double direct = triples / (1 << 20) * kDirect[op][mode != S2D_FP64][n_img % 3 != 0];
    return direct >= 118.0 + 0.45e-3 * (double)ns + 1e-3 * (double)nt + 0.6 * (double)ns / (double)nt;
}

bool far_possible(int mode, int64_t ns, int64_t nt) {
    for (int op = S2D_OP_SLP; op <= S2D_OP_SLP_TRACTION; ++op)
        if (far_worth(op, mode, ns, nt, 4, false)) return true;
    return false;
}

hipError_t far_setup(int op, const FarLayout &L, const s2d_curves *s, const s2d_targets *t, void *ws,
                     hipStream_t st) {
    char *b = (char *)ws;
    const int64_t N = L.ns + L.nt;
    double *box = (double *)(b + L.box);
    FarBox *info = (FarBox *)(box + 4 * kBoxBlocks);
    hipLaunchKernelGGL(far_box, dim3(kBoxBlocks), dim3(256), 0, st, L.ns, L.nt, s->x, s->y, t->x, t->y, box);
    hipLaunchKernelGGL(far_keys, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, st, L.ns, L.nt, s->x, s->y, t->x,
                       t->y, box, L.bits, info, (uint32_t *)(b + L.key[0]), (int32_t *)(b + L.idx[0]));
    for (int p = 0; 8 * p < L.bits; ++p) {
        const uint32_t *ki = (const uint32_t *)(b + L.key[p & 1]);
        const int32_t *xi = (const int32_t *)(b + L.idx[p & 1]);
        uint32_t *hist = (uint32_t *)(b + L.hist), *base = (uint32_t *)(b + L.base);
        hipLaunchKernelGGL(far_hist, dim3((unsigned)L.nblk), dim3(256), 0, st, N, L.nblk, 8 * p, ki, hist);
        hipLaunchKernelGGL(far_scan, dim3(64), dim3(256), 0, st, L.nblk, hist, base);
        hipLaunchKernelGGL(far_scatter, dim3((unsigned)L.nblk), dim3(256), 0, st, N, L.nblk, 8 * p, ki, xi, hist, base,
                           (uint32_t *)(b + L.key[(p + 1) & 1]), (int32_t *)(b + L.idx[(p + 1) & 1]));
    }
    FarNode *node = (FarNode *)(b + L.node);
    const int64_t ts = L.n0 / 2, tt = L.nT / 2;
    hipLaunchKernelGGL(far_tiles, dim3((unsigned)((ts + tt + 3) / 4)), dim3(256), 0, st, L.ns, L.nt, ts, tt, s->x,
                       s->y, t->x, t->y, (const int32_t *)(b + far_sorted(L)), (int32_t *)(b + L.spos), node,
                       (FarNode *)(b + L.tnode), (double *)(b + L.txy));
    hipLaunchKernelGGL(far_upper, dim3((unsigned)L.n2), dim3(64 * kFan), 0, st, L.n0, L.n1, node);
    if (op == S2D_OP_SLP && t->on_curve && s->n_curves > 0)
        hipLaunchKernelGGL(far_kress, dim3((unsigned)s->n_curves), dim3(256), 0, st, s->curve_off, s->n_curves, L.ns,
                           (double *)(b + L.kress));
    return hipGetLastError();
}

namespace {
template <int OP>
hipError_t far_sum_t(const FarLayout &L, const s2d_curves *s, const s2d_targets *t, const double *tnx,
                     const double *tny, double d, int32_t img_lo, int32_t img_hi, FinalArgs f, void *ws,
                     hipStream_t st) {
    char *b = (char *)ws;
    const int32_t *idx = (const int32_t *)(b + far_sorted(L));
    const FarNode *node = (const FarNode *)(b + L.node), *tnode = (const FarNode *)(b + L.tnode);
    const FarBox *info = (const FarBox *)((const double *)(b + L.box) + 4 * kBoxBlocks);
    const bool img0 = img_lo <= 0 && img_hi >= 0;
    double *coef = (double *)(b + L.coef), *txy = (double *)(b + L.txy), *part = (double *)(b + L.part);
    if (OP == S2D_OP_SLP && t->on_curve && img0) {
        double *self = (double *)(b + L.self);
        hipLaunchKernelGGL(far_self, dim3((unsigned)((L.nt + 255) / 256)), dim3(256), 0, st, L.nt, L.ns, t->on_curve,
                           t->on_node, s->curve_off, s->n_curves, s->nx, s->ny, s->w, s->fx, s->fy,
                           (const double *)(b + L.kress), self);
        f.self = self;
    } else {
        f.self = nullptr;
    }
    const P2mArgs pa{L.ns, L.n0, s->x, s->y, s->nx, s->ny, s->w, s->fx, s->fy, idx, node, info, b + L.rec, coef};
    constexpr int BASE = slp_sources(OP) ? S2D_OP_SLP : S2D_OP_DLP;
    hipLaunchKernelGGL(far_p2m<BASE>, dim3((unsigned)((L.n0 + 3) / 4)), dim3(256), 0, st, pa);
    hipLaunchKernelGGL(far_m2m, dim3((unsigned)L.n1), dim3(64 * kFan), 0, st, (int64_t)0, L.n0, kLeafFan, L.n0, node,
                       info, coef);
    hipLaunchKernelGGL(far_m2m, dim3((unsigned)L.n2), dim3(64 * kFan), 0, st, L.n0, L.n1, kFan, L.n0 + L.n1, node,
                       info, coef);
    const WalkArgs w{L.n0, L.n1, L.n2, node, d, img_lo, img_hi - img_lo + 1};
    const FarArgs fa{w, L.nt, tnode, info, coef, txy, part, idx + L.ns, tnx, tny};
    hipLaunchKernelGGL(far_far<OP>, dim3((unsigned)L.nT), dim3(64 * kFarWaves), 0, st, fa);
    const NearArgs na{w, L.ns, L.nt, L.groups, tnode, info, b + L.rec, txy, part, idx + L.ns,
                      (const int32_t *)(b + L.spos), img0 ? t->on_curve : nullptr, img0 ? t->on_node : nullptr, tnx, tny};
    hipLaunchKernelGGL(far_near<OP>, dim3((unsigned)(L.nT * L.groups)), dim3(64 * kNearWaves), 0, st, na, f);
    if (L.groups > 1)
        hipLaunchKernelGGL(far_final, dim3((unsigned)((L.nt + 255) / 256)), dim3(256), 0, st, L.nt, L.groups + 1, part,
                           idx + L.ns, f);
    return hipGetLastError();
}
}  // namespace

hipError_t far_sum(int op, const FarLayout &L, const s2d_curves *s, const s2d_targets *t, const double *tnx,
                   const double *tny, double d, int32_t img_lo, int32_t img_hi, FinalArgs f, void *ws,
                   hipStream_t st) {
    switch (op) {
    case S2D_OP_SLP: return far_sum_t<S2D_OP_SLP>(L, s, t, tnx, tny, d, img_lo, img_hi, f, ws, st);
    case S2D_OP_DLP: return far_sum_t<S2D_OP_DLP>(L, s, t, tnx, tny, d, img_lo, img_hi, f, ws, st);
    case S2D_OP_SLP_PRESSURE: return far_sum_t<S2D_OP_SLP_PRESSURE>(L, s, t, tnx, tny, d, img_lo, img_hi, f, ws, st);
    case S2D_OP_DLP_PRESSURE: return far_sum_t<S2D_OP_DLP_PRESSURE>(L, s, t, tnx, tny, d, img_lo, img_hi, f, ws, st);
    case S2D_OP_SLP_TRACTION: return far_sum_t<S2D_OP_SLP_TRACTION>(L, s, t, tnx, tny, d, img_lo, img_hi, f, ws, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace s2d
