// Spectral upsampling of periodic channel walls, the first step of the walls'
// close evaluation (the paper leaves close evaluation of the wall double
// layer to future work: Section 5 footnote; Section 6).
//
// Each wall curve is one period of a d-periodic wall with N (even, >= 4)
// nodes equispaced in its parameter t in [0, 2 pi), advancing by s d in x
// (s = +-1, from the first two nodes).  Its periodic parts x - s d t / 2 pi
// and y and the density are expanded in their discrete Fourier coefficients
// (stage 1) and evaluated at the P N parameter values 2 pi m / (P N) (stage 2,
// the trigonometric interpolant with the Nyquist mode split evenly between
// +-N/2), with spectral derivatives for the speed |x'(t)|, the weights
// (2 pi / P N) |x'| and the unit normals, oriented like the given normal of
// the coarse node at or before the fine one.
//
// Two routes, chosen per curve on the device (the sizes are known there only)
// by wall_factor: with N1 the largest divisor of N up to sqrt(N), N2 = N / N1,
//  * 8 (N1 + N2) < N and 20 (N1 + N2) < N + 500 + N^2 / 48,000, factored: the
//    series are the two complex ones (x - s d t / 2 pi) + i y and fx + i fy, fy
//    scaled to the size of fx; a transform of N points is N2 transforms of N1
//    points, a twiddle factor each, and N1 of N2 points, the fine points P shifted inverse transforms: N1 + N2 terms a value;
//  * otherwise (small N, a large prime factor), direct: coefficients V_k,
//    k = 0 .. N/2, as sums over the nodes and fine values as sums over the
//    modes, N/2 terms for four values at a time by symmetry.
// Both are chains of loads and multiply-adds: a factored value takes N1 + N2
// terms in turn, the direct route N^2 / 4 terms over the chip.  Kernel times of
// two walls refined 8 times, factored against direct at the same N, us: 300
// nodes (15 x 20) 37 / 35, 500 (20 x 25) 41 / 39, 1,000 (25 x 40) 47 / 46, 1,500
// (30 x 50) 53 / 58, 2,000 (40 x 50) 58 / 65, 2,500 (50 x 50) 63 / 72, 3,014 (22
// x 137) 86 / 84, 4,000 (50 x 80) 78 / 117, 7,940 (20 x 397) 250 / 290, 7,984 (16
// x 499) 300 / 294, 16,000 (125 x 128) 187 / 943.  Hence the second line; below
// 1,500 nodes the times are alike and the factored route's normals are three to
// ten times closer to the exact ones (4e-13 against 2e-12 at 2,352 nodes).
// Each kernel serves both routes, a curve's work-items leaving where the other
// route has them, so the factored one adds no launch; its loops are kept to the
// registers of the direct route's (124 and 126 in the first and third kernel:
// with 211 and 192 the direct route took 1.2-1.45 times as long).
// At 16,000 nodes its kernels (12, 26, 24, 58 and 68 us) wait for the caches:
// 500 waves in stage 1, 75 MB of intermediate sums read 64 times over in the
// last, which takes two outputs from each.
//
// Direct route: coefficients are stored interleaved, 8 doubles per (curve, k):
// re and im of the four series.  Both sums are split into chunks (over the
// nodes in stage 1, over the modes in stage 2) along the grid's y dimension so
// that the launch fills the device, and the chunks' partial sums are added in
// chunk order by a second kernel (deterministic results).  A wave whose lanes
// all lie in one curve reads the coefficients (and in stage 1 the nodes)
// through the scalar data path.  Twiddle factors follow a rotation recurrence
// re-anchored with sincospi every 32 steps (16 on the factored route).
//
// The factored route keeps its sums inside the curve's own share of the direct
// one's scratch: stage 1 in the first chunk's records (4 of 8 doubles), the
// coefficients in the curve's records (4 of 8), stage 2 in the first chunk's
// six arrays, and N1 and fy's factor in doubles 4 .. 6 of the curve's
// last record, which the direct route (k <= N/2 < N - 1) leaves alone.
#include "s2d_near.h"

#include <algorithm>

namespace s2d {

namespace {

constexpr int kAnchor = 32;
constexpr int kTurn = 16;

struct alignas(16) Coef8 { double v[8]; };        // (re, im) of x~, y, fx, fy

// element i of a device array, read through the constant address space (the
// scalar path when the address is wave-uniform), one dword at a time
template <class T>
__device__ __forceinline__ T load_ro(const void *base, int64_t i) {
    constexpr int n = (int)(sizeof(T) / 4);
    using CP = const __attribute__((address_space(4))) uint32_t *;
    const CP p = (CP)((const char *)base + i * (int64_t)sizeof(T));
    struct Words { uint32_t w[n]; } t;
#pragma unroll
    for (int k = 0; k < n; ++k) t.w[k] = p[k];
    return __builtin_bit_cast(T, t);
}

template <bool UNI, class T>
__device__ __forceinline__ T ld(const T *p, int64_t i) {
    if constexpr (UNI) return load_ro<T>(p, i);
    else return p[i];
}

// the curve c with off[c] * scale <= g < off[c + 1] * scale (off ascending)
__device__ __forceinline__ int find_curve(const int32_t *__restrict__ off, int n, int64_t g, int64_t scale) {
    int lo = 0, hi = n;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if ((int64_t)off[mid] * scale <= g) lo = mid; else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ bool curve_ok(int64_t lo, int64_t hi, int64_t n_nodes) {
    return lo >= 0 && hi <= n_nodes && hi - lo >= 4 && ((hi - lo) & 1) == 0;
}

// e^{2 pi i num / den}, 0 <= num < den
struct Cx { double r, i; };
// a call of its own: sincospi inlined for every factor keeps them all in registers
__device__ __noinline__ Cx root(uint32_t num, uint32_t den) {
    Cx z;
    sincospi(2.0 * (double)num / (double)den, &z.i, &z.r);
    return z;
}
__device__ __forceinline__ Cx mul(Cx a, Cx b) { return {a.r * b.r - a.i * b.i, a.r * b.i + a.i * b.r}; }

// use(a, e^{2 pi i (base + a step) / den}, load(a)) for a = a0 .. a1-1 (0 <= base,
// step < den), the loads of four terms issued together (past the end: zero
// terms): one term's at a time wait for a cache miss each, and eight terms' at a
// time take registers that the direct route's kernels pay for (two waves a SIMD
// instead of four: 1.24-1.33 times their time).  A term's factor is at most
// five products away from sincospi values (a chain over 32 terms doubles the
// error of the derivatives).
template <class L, class F>
__device__ __forceinline__ void rotate(int a0, int a1, uint32_t base, uint32_t step, uint32_t den, L &&load, F &&use) {
    if (a0 >= a1) return;
    Cx w1 = root(step, den), w2 = root((uint32_t)(2ull * step % den), den), w4 = root((uint32_t)(4ull * step % den), den);
    for (int s0 = a0; s0 < a1; s0 += kTurn) {
        Cx z = root((uint32_t)((base + (uint64_t)s0 * step) % den), den);
        const int s1 = min(s0 + kTurn, a1);
        for (int a = s0; a < s1; a += 4) {
            double4 v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = load(min(a + e, s1 - 1));
            const double4 none{0.0, 0.0, 0.0, 0.0};
            use(a, z, v[0]);
            use(a + 1, mul(z, w1), a + 1 < s1 ? v[1] : none);
            const Cx y = mul(z, w2);
            use(a + 2, y, a + 2 < s1 ? v[2] : none);
            use(a + 3, mul(y, w1), a + 3 < s1 ? v[3] : none);
            z = mul(z, w4);
        }
    }
}

// Whether N = N1 N2 nodes are factored: never up to kFactorMin, as
// N1 + N2 >= 2 sqrt(N).
constexpr int64_t kFactorMin = 256;
__device__ __forceinline__ bool pays(uint64_t N1, uint64_t N) {
    const uint64_t s = N1 + N / N1;
    return 8 * s < N && 20 * s < N + 500 + N * N / 48000;
}

// What wall_factor leaves in doubles 4 .. 6 of the curve's last record: N1 (0:
// direct route), the factor that brings fy to fx's size (a power of two; 0: fy
// is zero throughout), and 0 where fx is zero throughout, else 1.
struct Factored { double n1, rf, on; };
__device__ __forceinline__ Factored factored(const WallArgs &a, int64_t lo, int64_t N) {
    const double *v = ((const Coef8 *)a.coef)[lo + N - 1].v + 4;
    return Factored{v[0], v[1], v[2]};
}
__device__ __forceinline__ int factor_of(const WallArgs &a, int64_t lo, int64_t N) {
    if (a.n_nodes <= kFactorMin) return 0;              // no curve can be factored
    const int n1 = (int)((const Coef8 *)a.coef)[lo + N - 1].v[4];
    return n1 >= 2 && N % n1 == 0 ? n1 : 0;
}

// node g = lo + j relative to the curve's first node, x without its advance
__device__ __forceinline__ double4 wall_series(const WallArgs &a, int64_t lo, int64_t j, double sd) {
    const int64_t g = lo + j;
    return double4{(a.x[g] - a.x[lo]) - sd * (double)j, a.y[g] - a.y[lo], a.fx[g], a.fy[g]};
}

// orders magnitudes; 0 for zero, 0x7ff00000 and above for what is not finite
__device__ __forceinline__ uint32_t size_key(double v) {
    return ((uint32_t)__double2hiint(v) & 0x7fffffffu) | (__double2loint(v) != 0 ? 1u : 0u);
}

// A workgroup per curve: N1, fy's factor, and the fine curve's offset where one
// is asked for.  A complex series leaves rounding of its larger component in
// the smaller one and a value that is not finite in both: fy comes in at fx's
// size, and curves with such values, or with sizes 2^500 apart, take the direct
// route.  (x and y stay as they are: their errors meet in one length, and x's
// periodic part may be mere rounding, white up to the modes that a derivative
// magnifies; brought to one size with y it trebles the normals' error.)
__global__ __launch_bounds__(1024) void wall_factor(WallArgs a) {
    __shared__ uint32_t top[4];
    const int c = blockIdx.x, lane = threadIdx.x & (kWave - 1);
    const int64_t lo = a.off[c];
    if (a.ooff && threadIdx.x == 0) a.ooff[c] = (int32_t)lo * a.P;
    if (c == a.n_curves) return;
    const int64_t hi = a.off[c + 1];
    if (a.n_nodes <= kFactorMin || !curve_ok(lo, hi, a.n_nodes)) return;
    const uint32_t N = (uint32_t)(hi - lo);
    uint32_t best = 1;
    for (uint64_t t = 2 + lane; t * t <= N; t += kWave)
        if (N % (uint32_t)t == 0) best = (uint32_t)t;
#pragma unroll
    for (int m = kWave / 2; m >= 1; m >>= 1) best = max(best, (uint32_t)__shfl_xor((int)best, m, kWave));
    double *o = ((Coef8 *)a.coef)[hi - 1].v + 4;
    if (!pays(best, N)) {                               // the same for all threads
        if (threadIdx.x == 0) o[0] = 0.0;
        return;
    }
    if (threadIdx.x < 4) top[threadIdx.x] = 0;
    __syncthreads();
    const double sd = (a.x[lo + 1] > a.x[lo] ? 1.0 : -1.0) * a.d / (double)N;
    uint32_t k[4] = {0, 0, 0, 0};
#pragma unroll 4
    for (int64_t j = threadIdx.x; j < N; j += 1024) {
        const double4 v = wall_series(a, lo, j, sd);
        k[0] = max(k[0], size_key(v.x));
        k[1] = max(k[1], size_key(v.y));
        k[2] = max(k[2], size_key(v.z));
        k[3] = max(k[3], size_key(v.w));
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int m = kWave / 2; m >= 1; m >>= 1) k[q] = max(k[q], (uint32_t)__shfl_xor((int)k[q], m, kWave));
        if (lane == 0) atomicMax(&top[q], k[q]);
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    const int e = (int)(top[2] >> 20) - (int)(top[3] >> 20);
    const bool fit = max(max(top[0], top[1]), max(top[2], top[3])) < 0x7ff00000u &&
                     (top[2] == 0 || top[3] == 0 || abs(e) <= 500);
    o[0] = fit ? (double)best : 0.0;
    o[1] = top[3] == 0 ? 0.0 : top[2] == 0 ? 1.0 : ldexp(1.0, e);
    o[2] = top[2] == 0 ? 0.0 : 1.0;
}

// Z += (v.x + i v.y) z, F += (v.z + i v.w) z
__device__ __forceinline__ void add_turned(Cx &Z, Cx &F, Cx z, double4 v) {
    Z.r = __builtin_fma(v.x, z.r, __builtin_fma(-v.y, z.i, Z.r));
    Z.i = __builtin_fma(v.x, z.i, __builtin_fma(v.y, z.r, Z.i));
    F.r = __builtin_fma(v.z, z.r, __builtin_fma(-v.w, z.i, F.r));
    F.i = __builtin_fma(v.z, z.i, __builtin_fma(v.w, z.r, F.i));
}

// Factored stage 1, item l = b N1 + k1: sum over a of the values at node
// N2 a + b (positions relative to the first node: y's mean would leave its
// rounding in x) times e^{-2 pi i a k1 / N1}, and the twiddle factor e^{-2 pi i b k1 / N}
__device__ __forceinline__ void factored_dft_a(const WallArgs &a, int64_t lo, int64_t N, int N1, int64_t l, double s) {
    const int N2 = (int)((uint32_t)N / (uint32_t)N1), b = (int)((uint32_t)l / (uint32_t)N1), k1 = (int)l - b * N1;
    const double sd = s * a.d / (double)N;
    const double rf = factored(a, lo, N).rf;
    Cx Z{0, 0}, F{0, 0};
    rotate(
        0, N1, 0, (N1 - k1) % N1, N1,
        [&](int i) {
            double4 v = wall_series(a, lo, (int64_t)N2 * i + b, sd);
            v.w *= rf;
            return v;
        },
        [&](int, Cx z, double4 v) { add_turned(Z, F, z, v); });
    const uint32_t n = (uint32_t)N, turn = (uint32_t)b * (uint32_t)k1;      // b k1 < N
    const Cx t = root(turn ? n - turn : 0, n);
    Z = mul(Z, t);
    F = mul(F, t);
    double4 *o = (double4 *)(((Coef8 *)a.part1)[lo + l].v);
    *o = double4{Z.r, Z.i, F.r, F.i};
}

// and item k = k1 + N1 k2: coefficient k of both complex series
__device__ __forceinline__ void factored_dft_b(const WallArgs &a, int64_t lo, int64_t N, int N1, int64_t k) {
    const int N2 = (int)((uint32_t)N / (uint32_t)N1), k2 = (int)((uint32_t)k / (uint32_t)N1), k1 = (int)k - k2 * N1;
    const Coef8 *T = (const Coef8 *)a.part1 + lo + k1;
    Cx Z{0, 0}, F{0, 0};
    rotate(
        0, N2, 0, (N2 - k2) % N2, N2, [&](int b) { return *(const double4 *)T[(int64_t)b * N1].v; },
        [&](int, Cx z, double4 v) { add_turned(Z, F, z, v); });
    *(double4 *)((Coef8 *)a.coef)[lo + k].v = double4{Z.r, Z.i, F.r, F.i};
}

// Factored stage 2 at the shift r / P of a node spacing, item l = b N1 + k1:
// sum over a of the coefficients k = N2 a + b (frequency k below N/2, k - N
// above) of the first series, its derivative and the second, times
// e^{2 pi i a (P k1 + r) / (P N1)} (less r / P of a turn above N/2), and
// e^{2 pi i b (P k1 + r) / (P N)}; the Nyquist term by cos(pi r / P), its
// derivative by -N/2 sin(pi r / P), times (-1)^q at node q
__device__ __forceinline__ void factored_synth_a(const WallArgs &a, int64_t lo, int64_t N, int N1, int r, int64_t l) {
    const int N2 = (int)((uint32_t)N / (uint32_t)N1), b = (int)((uint32_t)l / (uint32_t)N1), k1 = (int)l - b * N1;
    const int h = (int)(N / 2);
    const int64_t P = a.P, step = P * k1 + r;
    const Coef8 *coef = (const Coef8 *)a.coef + lo;
    Cx Z{0, 0}, D{0, 0}, F{0, 0};
    const auto load = [&](int i) { return *(const double4 *)coef[N2 * i + b].v; };
    const auto add = [&](double kd, Cx z, double4 v) {
        const double pr = __builtin_fma(v.x, z.r, -v.y * z.i), pi = __builtin_fma(v.x, z.i, v.y * z.r);
        Z.r += pr;
        Z.i += pi;
        D.r = __builtin_fma(-kd, pi, D.r);
        D.i = __builtin_fma(kd, pr, D.i);
        F.r = __builtin_fma(v.z, z.r, __builtin_fma(-v.w, z.i, F.r));
        F.i = __builtin_fma(v.z, z.i, __builtin_fma(v.w, z.r, F.i));
    };
    // k = N2 i + b < h for i < i0, > h for i >= i1
    const int i0 = b < h ? (h - b + N2 - 1) / N2 : 0, i1 = b <= h ? (h - b) / N2 + 1 : 0;
    rotate(0, i0, 0, step, P * N1, load, [&](int i, Cx z, double4 v) { add((double)(N2 * i + b), z, v); });
    rotate(i1, N1, (P - r) % P * N1, step, P * N1, load,
           [&](int i, Cx z, double4 v) { add((double)(N2 * i + b) - (double)N, z, v); });
    const Cx t = root((int64_t)b * step % (P * N), P * N);
    Z = mul(Z, t);
    D = mul(D, t);
    F = mul(F, t);
    if (i0 < i1) {                                      // h = N2 i0 + b
        const double4 v = *(const double4 *)coef[h].v;
        double sn, cs;
        sincospi((double)r / (double)P, &sn, &cs);
        const double e = (k1 & 1) ? -1.0 : 1.0, c = e * cs, ds = -e * (double)h * sn;   // e^{2 pi i h k1 / N}
        Z.r = __builtin_fma(c, v.x, Z.r);
        Z.i = __builtin_fma(c, v.y, Z.i);
        D.r = __builtin_fma(ds, v.x, D.r);
        D.i = __builtin_fma(ds, v.y, D.i);
        F.r = __builtin_fma(c, v.z, F.r);
        F.i = __builtin_fma(c, v.w, F.i);
    }
    const int64_t nf = P * a.n_nodes;
    double *o = a.part2 + P * (lo + l) + r;             // shifts side by side: the next step's lanes
    o[0] = Z.r;
    o[nf] = Z.i;
    o[2 * nf] = F.r;
    o[3 * nf] = F.i;
    o[4 * nf] = D.r;
    o[5 * nf] = D.i;
}

// stage 1 sums for coefficient k of the curve at lo with N nodes, over its
// nodes jb .. je-1
template <bool UNI>
__device__ __forceinline__ void dft_sums(const WallArgs &a, int64_t lo, int64_t N, int64_t k, int64_t jb,
                                         int64_t je, double s, double re[4], double im[4]) {
    double wr, wi;
    sincospi(2.0 * (double)k / (double)N, &wi, &wr);
    wi = -wi;                                           // e^{-2 pi i k / N}
    const double sd = s * a.d / (double)N;
    for (int64_t j0 = jb; j0 < je; j0 += kAnchor) {
        double zr, zi;
        sincospi(2.0 * (double)((j0 * k) % N) / (double)N, &zi, &zr);
        zi = -zi;
        const int64_t j1 = min(j0 + (int64_t)kAnchor, je);
        for (int64_t j = j0; j < j1; ++j) {
            const double v[4] = {ld<UNI>(a.x, lo + j) - sd * (double)j, ld<UNI>(a.y, lo + j), ld<UNI>(a.fx, lo + j),
                                 ld<UNI>(a.fy, lo + j)};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                re[q] = __builtin_fma(v[q], zr, re[q]);
                im[q] = __builtin_fma(v[q], zi, im[q]);
            }
            const double tr = zr * wr - zi * wi;
            zi = zr * wi + zi * wr;
            zr = tr;
        }
    }
}

// stage 1, split over the nodes: work-item g, chunk blockIdx.y ->
// coefficient k = g - off[c] of curve c (k <= N/2) over the chunk's nodes
__global__ __launch_bounds__(256) void wall_dft_part(WallArgs a) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= a.n_nodes) return;
    const int c = find_curve(a.off, a.n_curves, g, 1);
    const int64_t lo = a.off[c], hi = a.off[c + 1], N = hi - lo, k = g - lo;
    if (!curve_ok(lo, hi, a.n_nodes) || k < 0 || k >= N) return;
    const int N1 = factor_of(a, lo, N);
    if (N1 ? blockIdx.y > 0 : k > N / 2) return;
    const double s = a.x[lo + 1] > a.x[lo] ? 1.0 : -1.0;
    if (N1) {
        factored_dft_a(a, lo, N, N1, k, s);
        return;
    }
    const int64_t S = a.s1, sc = blockIdx.y, len = (N + S - 1) / S;
    const int64_t jb = min(sc * len, N), je = min(jb + len, N);
    double re[4] = {0, 0, 0, 0}, im[4] = {0, 0, 0, 0};
    const int lo_u = __builtin_amdgcn_readfirstlane((int)lo);
    if (__all(lo == (int64_t)lo_u)) {
        // one curve: N and the chunk bounds are wave-uniform (scalar loop,
        // scalar loads of the nodes)
        const int N_u = __builtin_amdgcn_readfirstlane((int)N);
        const int jb_u = __builtin_amdgcn_readfirstlane((int)jb), je_u = __builtin_amdgcn_readfirstlane((int)je);
        dft_sums<true>(a, lo_u, N_u, k, jb_u, je_u, s, re, im);
    } else {
        dft_sums<false>(a, lo, N, k, jb, je, s, re, im);
    }
    Coef8 o;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        o.v[2 * q] = re[q];
        o.v[2 * q + 1] = im[q];
    }
    ((Coef8 *)a.part1)[sc * a.n_nodes + lo + k] = o;
}

// the chunks' partial coefficients summed in chunk order; the factored
// route's second step
__global__ __launch_bounds__(256) void wall_dft_sum(WallArgs a) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= a.n_nodes) return;
    const int c = find_curve(a.off, a.n_curves, g, 1);
    const int64_t lo = a.off[c], hi = a.off[c + 1], N = hi - lo, k = g - lo;
    if (!curve_ok(lo, hi, a.n_nodes) || k < 0 || k >= N) return;
    const int N1 = factor_of(a, lo, N);
    if (N1) {
        factored_dft_b(a, lo, N, N1, k);
        return;
    }
    if (k > N / 2) return;
    const Coef8 *p = (const Coef8 *)a.part1;
    Coef8 o = p[g];
    for (int sc = 1; sc < a.s1; ++sc) {
        const Coef8 t = p[(int64_t)sc * a.n_nodes + g];
#pragma unroll
        for (int q = 0; q < 8; ++q) o.v[q] += t.v[q];
    }
    ((Coef8 *)a.coef)[g] = o;
}

// stage 2 sums over modes k = kb .. ke-1 at the fine angle th = 2 pi j / M,
// kept apart by the parity of k - kb (A: even, B: odd) and split into
// C = sum Re V_k cos k th, S = sum Im V_k sin k th (four series) and
// DS = sum k Re V_k sin k th, DC = sum k Im V_k cos k th (x~ and y only).
// Then Re sum V_k e^{ik th} = C - S and Re sum i k V_k e^{ik th} = -(DS + DC);
// at -th the sine parts change sign, and at th + pi the odd-k parts do.
struct SynthAcc { double C[4], S[4], DS[2], DC[2]; };

template <bool UNI>
__device__ __forceinline__ void synth_step(const Coef8 *coef, int64_t lo, int64_t k, double zr, double zi,
                                           SynthAcc &X) {
    const Coef8 V = ld<UNI>(coef, lo + k);
    const double kd = (double)k;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        X.C[q] = __builtin_fma(V.v[2 * q], zr, X.C[q]);
        X.S[q] = __builtin_fma(V.v[2 * q + 1], zi, X.S[q]);
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        X.DS[q] = __builtin_fma(kd * V.v[2 * q], zi, X.DS[q]);
        X.DC[q] = __builtin_fma(kd * V.v[2 * q + 1], zr, X.DC[q]);
    }
}

template <bool UNI>
__device__ __forceinline__ void synth_sums(const Coef8 *coef, int64_t lo, int64_t kb, int64_t ke, int64_t j,
                                           int64_t M, SynthAcc &A, SynthAcc &B) {
    double wr, wi;
    sincospi(2.0 * (double)j / (double)M, &wi, &wr);   // e^{i th}
    for (int64_t k0 = kb; k0 < ke; k0 += kAnchor) {      // kAnchor is even: k0 - kb stays even
        double zr, zi;
        sincospi(2.0 * (double)((k0 * j) % M) / (double)M, &zi, &zr);
        const int64_t k1 = min(k0 + (int64_t)kAnchor, ke);
        int64_t k = k0;
        for (; k + 1 < k1; k += 2) {
            synth_step<UNI>(coef, lo, k, zr, zi, A);
            double tr = zr * wr - zi * wi;
            zi = zr * wi + zi * wr;
            zr = tr;
            synth_step<UNI>(coef, lo, k + 1, zr, zi, B);
            tr = zr * wr - zi * wi;
            zi = zr * wi + zi * wr;
            zr = tr;
        }
        if (k < k1) synth_step<UNI>(coef, lo, k, zr, zi, A);
    }
}

// stage 2, split over the modes 1 .. h-1: work-item g, chunk blockIdx.y.
// Curve c owns the P N / 2 work-items from ceil(P off[c] / 2); item j <= M / 4
// of the curve serves the fine points j, M - j, M/2 + j and M/2 - j (the
// rest return at once).  Six partial sums per fine point and chunk.  Factored
// curves: work-item t of chunk y takes item t + y times the curve's work-items.
__global__ __launch_bounds__(256) void wall_synth_part(WallArgs a) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t P = a.P, nf = P * a.n_nodes;
    if (2 * g >= nf) return;
    const int c = find_curve(a.off, a.n_curves, 2 * g, P);
    const int64_t lo = a.off[c], hi = a.off[c + 1], N = hi - lo, M = P * N, h = N / 2;
    const int64_t j = g - (P * lo + 1) / 2;
    if (!curve_ok(lo, hi, a.n_nodes) || j < 0) return;
    const int N1 = factor_of(a, lo, N);
    if (N1) {
        const int64_t m = j + blockIdx.y * h * P;
        if (j < h * P && m < M) factored_synth_a(a, lo, N, N1, (int)((uint32_t)m % (uint32_t)P), (uint32_t)m / (uint32_t)P);
        return;
    }
    if (j > M / 4 || blockIdx.y >= a.s2) return;
    const int64_t S = a.s2, sc = blockIdx.y, len = (h - 1 + S - 1) / S;
    const int64_t kb = min(1 + sc * len, h), ke = min(kb + len, h);
    const Coef8 *coef = (const Coef8 *)a.coef;
    SynthAcc A = {}, B = {};
    const int lo_u = __builtin_amdgcn_readfirstlane((int)lo);
    if (__all(lo == (int64_t)lo_u)) {
        // one curve: the mode range is wave-uniform (scalar loop, scalar
        // loads of the coefficients)
        const int kb_u = __builtin_amdgcn_readfirstlane((int)kb), ke_u = __builtin_amdgcn_readfirstlane((int)ke);
        synth_sums<true>(coef, lo_u, kb_u, ke_u, j, M, A, B);
    } else {
        synth_sums<false>(coef, lo, kb, ke, j, M, A, B);
    }
    const bool odd = kb & 1;                            // A holds the odd k when kb is odd
    SynthAcc E, O;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        E.C[q] = odd ? B.C[q] : A.C[q];
        O.C[q] = odd ? A.C[q] : B.C[q];
        E.S[q] = odd ? B.S[q] : A.S[q];
        O.S[q] = odd ? A.S[q] : B.S[q];
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        E.DS[q] = odd ? B.DS[q] : A.DS[q];
        O.DS[q] = odd ? A.DS[q] : B.DS[q];
        E.DC[q] = odd ? B.DC[q] : A.DC[q];
        O.DC[q] = odd ? A.DC[q] : B.DC[q];
    }
    const int64_t pts[4] = {j, j ? M - j : 0, M / 2 + j, M / 2 - j};
    double *base = a.part2 + sc * 6 * nf + P * lo;
#pragma unroll
    for (int o = 0; o < 4; ++o) {
        const double ho = (o & 2) ? -1.0 : 1.0, rs = (o & 1) ? -1.0 : 1.0;
        double *p = base + pts[o];
#pragma unroll
        for (int q = 0; q < 4; ++q) p[q * nf] = (E.C[q] + ho * O.C[q]) - rs * (E.S[q] + ho * O.S[q]);
#pragma unroll
        for (int q = 0; q < 2; ++q) p[(4 + q) * nf] = -rs * (E.DS[q] + ho * O.DS[q]) - (E.DC[q] + ho * O.DC[q]);
    }
}

// node, normal, weight and density of fine point m of the curve at lo from
// the four series' values and the first two's derivatives
__device__ __forceinline__ void fine_point(const WallArgs &a, int64_t lo, int64_t M, int64_t m, double s,
                                           const double val[4], const double der[2]) {
    const int64_t g = a.P * lo + m, j = lo + m / a.P;
    const double dX = der[0] + s * a.d / (2.0 * M_PI), dY = der[1];
    const double sp = sqrt(dX * dX + dY * dY);
    const double o = (-dY * a.nx[j] + dX * a.ny[j]) > 0.0 ? 1.0 : -1.0;
    a.ox[g] = val[0] + s * a.d * ((double)m / (double)M);
    a.oy[g] = val[1];
    a.onx[g] = -o * dY / sp;
    a.ony[g] = o * dX / sp;
    a.ow[g] = (2.0 * M_PI / (double)M) * sp;
    a.ofx[g] = val[2];
    a.ofy[g] = val[3];
}

// Factored stage 2, last step, item t = (g N1 + k1) P + r: fine points
// P (k1 + N1 k2) + r for k2 = OUT g .. OUT g + OUT - 1, the sums over b of stage
// 2's first step times e^{2 pi i b k2 / N2}, BATCH terms' loads at a time.  Two
// outputs share each load; one in eights halves the chain of loads where the
// launch leaves the chip room (up to kRound fine points: two waves a SIMD).
constexpr int64_t kRound = 131072;
template <int OUT, int BATCH>
__device__ __forceinline__ void factored_synth_b(const WallArgs &a, int64_t lo, int64_t N, int N1, int64_t t, double s) {
    const int64_t P = a.P, M = P * N, nf = P * a.n_nodes;
    const uint32_t N2 = (uint32_t)N / (uint32_t)N1, P32 = (uint32_t)P, tp = (uint32_t)t / P32;
    const uint32_t r = (uint32_t)t - tp * P32, g = tp / (uint32_t)N1, k1 = tp - g * (uint32_t)N1;
    if (OUT * g >= N2) return;
    const double *T = a.part2 + P * (lo + k1) + r;
    const int64_t row = P * N1;
    double acc[OUT][6] = {};
    // factors as in rotate()
    const auto turned = [&](uint64_t num) { return root((uint32_t)(num % N2), N2); };
    Cx w1[OUT], w2[OUT], w4[OUT], wb[OUT], z[OUT];
    uint32_t k2[OUT];
#pragma unroll
    for (int e = 0; e < OUT; ++e) {
        k2[e] = min(OUT * g + e, N2 - 1);
        w1[e] = turned(k2[e]);
        w2[e] = turned(2ull * k2[e]);
        w4[e] = turned(4ull * k2[e]);
        wb[e] = BATCH == 4 ? w4[e] : turned((uint64_t)BATCH * k2[e]);
    }
    for (uint32_t b0 = 0; b0 < N2; b0 += BATCH) {
        if (b0 % kTurn == 0) {
#pragma unroll
            for (int e = 0; e < OUT; ++e) z[e] = turned((uint64_t)b0 * k2[e]);
        }
        double v[BATCH][6];
#pragma unroll
        for (int f = 0; f < BATCH; ++f) {
            const double *p = T + (int64_t)min(b0 + f, N2 - 1) * row;
#pragma unroll
            for (int q = 0; q < 6; ++q) v[f][q] = p[q * nf];
        }
#pragma unroll
        for (int e = 0; e < OUT; ++e) {
            Cx y[BATCH];
            y[0] = z[e];
#pragma unroll
            for (int f = 1; f < BATCH; ++f) y[f] = f == 4 ? mul(z[e], w4[e]) : (f & 1) ? mul(y[f - 1], w1[e]) : mul(y[f - 2], w2[e]);
#pragma unroll
            for (int f = 0; f < BATCH; ++f) {
                const bool in = b0 + f < N2;
                const double yr = in ? y[f].r : 0.0, yi = in ? y[f].i : 0.0;
#pragma unroll
                for (int q = 0; q < 6; q += 2) {
                    acc[e][q] = __builtin_fma(v[f][q], yr, __builtin_fma(-v[f][q + 1], yi, acc[e][q]));
                    acc[e][q + 1] = __builtin_fma(v[f][q], yi, __builtin_fma(v[f][q + 1], yr, acc[e][q + 1]));
                }
            }
            z[e] = mul(z[e], wb[e]);
        }
    }
    const double invN = 1.0 / (double)N;
    const Factored fac = factored(a, lo, N);
    // a component that is zero stays an exact zero
    const double outx = fac.on * invN, outy = fac.rf != 0.0 ? invN * (1.0 / fac.rf) : 0.0;
#pragma unroll
    for (int e = 0; e < OUT; ++e) {
        if (OUT * g + e >= N2) return;
#pragma unroll
        for (int q = 0; q < 6; ++q) acc[e][q] *= q == 2 ? outx : q == 3 ? outy : invN;
        acc[e][0] += a.x[lo];
        acc[e][1] += a.y[lo];
        fine_point(a, lo, M, P * (k1 + (int64_t)N1 * k2[e]) + r, s, acc[e], acc[e] + 4);
    }
}

// stage 2 finish: the chunks' sums in chunk order, the mean and Nyquist
// terms, then fine point g; the factored route's last step
__global__ __launch_bounds__(256) void wall_synth_fin(WallArgs a) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t P = a.P, nf = P * a.n_nodes;
    if (g >= nf) return;
    const int c = find_curve(a.off, a.n_curves, g, P);
    const int64_t lo = a.off[c], hi = a.off[c + 1], N = hi - lo, M = P * N, m = g - P * lo, h = N / 2;
    if (!curve_ok(lo, hi, a.n_nodes) || m < 0 || m >= M) {
        const double nan = __builtin_nan("");
        a.ox[g] = a.oy[g] = a.onx[g] = a.ony[g] = a.ow[g] = a.ofx[g] = a.ofy[g] = nan;
        return;
    }
    const double s = a.x[lo + 1] > a.x[lo] ? 1.0 : -1.0;
    const int N1 = factor_of(a, lo, N);
    if (N1) {
        if (nf <= kRound)
            factored_synth_b<1, 8>(a, lo, N, N1, m, s);
        else
            factored_synth_b<2, 4>(a, lo, N, N1, m, s);
        return;
    }
    double acc[4] = {0, 0, 0, 0}, dac[2] = {0, 0};
    for (int sc = 0; sc < a.s2; ++sc) {
        const double *p = a.part2 + (int64_t)sc * 6 * nf + g;
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] += p[q * nf];
        dac[0] += p[4 * nf];
        dac[1] += p[5 * nf];
    }
    const Coef8 *coef = (const Coef8 *)a.coef;
    const Coef8 V0 = coef[lo], Vh = coef[lo + h];
    double sh, ch;
    sincospi(2.0 * (double)((h * m) % M) / (double)M, &sh, &ch);
    const double invN = 1.0 / (double)N;
    double val[4], der[2];
#pragma unroll
    for (int q = 0; q < 4; ++q) val[q] = (V0.v[2 * q] + 2.0 * acc[q] + Vh.v[2 * q] * ch) * invN;
#pragma unroll
    for (int q = 0; q < 2; ++q) der[q] = (2.0 * dac[q] - (double)h * Vh.v[2 * q] * sh) * invN;
    fine_point(a, lo, M, m, s, val, der);
}

// u (+)= uf - uc, v (+)= vf - vc: the difference is rounded first, so an
// accumulated result equals the written one added to the prior contents
__global__ __launch_bounds__(256) void delta_combine(int64_t n, int acc, double *__restrict__ u,
                                                     double *__restrict__ v, const double *__restrict__ t) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double du = t[i] - t[2 * n + i], dv = t[n + i] - t[3 * n + i];
    u[i] = acc ? u[i] + du : du;
    v[i] = acc ? v[i] + dv : dv;
}

__global__ __launch_bounds__(256) void add_or_write(int64_t n, int acc, double *__restrict__ u,
                                                    double *__restrict__ v, const double *__restrict__ tu,
                                                    const double *__restrict__ tv) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    u[i] = acc ? u[i] + tu[i] : tu[i];
    v[i] = acc ? v[i] + tv[i] : tv[i];
}

// one vector atomic per fallback target
__global__ __launch_bounds__(256) void fallback_compact(int64_t n, const int32_t *__restrict__ flag,
                                                        const double *__restrict__ tx, const double *__restrict__ ty,
                                                        int32_t *__restrict__ list, int32_t *__restrict__ count,
                                                        double *__restrict__ cx, double *__restrict__ cy) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n || flag[i] != 1) return;
    const int32_t j = atomicAdd(count, 1);
    list[j] = (int32_t)i;
    cx[j] = tx[i];
    cy[j] = ty[i];
}

__global__ __launch_bounds__(256) void fallback_scatter(int64_t m, const int32_t *__restrict__ list,
                                                        const double *__restrict__ t4, double *__restrict__ tu,
                                                        double *__restrict__ tv) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= m) return;
    const int32_t i = list[j];
    tu[i] = t4[j] - t4[2 * m + j];
    tv[i] = t4[m + j] - t4[3 * m + j];
}

__global__ void zero_int(int32_t *p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

unsigned grid(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

void wall_splits(int64_t n_nodes, int P, int *s1, int *s2) {
    // chunks enough for about 8 (stage 1) and 16 (stage 2) waves per SIMD
    // of a 256-CU device; more work per chunk than that gains nothing
    constexpr int64_t kItems1 = 256LL * 4 * 8 * 64, kItems2 = 2 * kItems1;
    const int64_t n1 = std::max<int64_t>(n_nodes, 1), n2 = std::max<int64_t>((int64_t)P * n_nodes, 1);
    *s1 = (int)std::min<int64_t>(std::max<int64_t>((kItems1 + n1 - 1) / n1, 1), 32);
    *s2 = (int)std::min<int64_t>(std::max<int64_t>((kItems2 + n2 - 1) / n2, 1), 16);
}

WallScratch wall_scratch(int64_t n_nodes, int P) {
    WallScratch w{};
    wall_splits(n_nodes, P, &w.s1, &w.s2);
    const auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    w.coef = 0;
    w.part1 = al((size_t)n_nodes * sizeof(Coef8));
    w.part2 = w.part1 + al((size_t)w.s1 * n_nodes * sizeof(Coef8));
    w.total = w.part2 + al((size_t)w.s2 * 6 * P * n_nodes * sizeof(double));
    return w;
}

hipError_t wall_upsample_launch(const WallArgs &a, hipStream_t st) {
    if (a.n_curves > 0 && a.off)
        hipLaunchKernelGGL(wall_factor, dim3((unsigned)a.n_curves + 1),
                           dim3(a.n_nodes <= kFactorMin ? kWave : 1024), 0, st, a);
    if (a.n_nodes > 0) {
        const unsigned g1 = grid(a.n_nodes), g2 = grid(((int64_t)a.P * a.n_nodes + 1) / 2);
        hipLaunchKernelGGL(wall_dft_part, dim3(g1, (unsigned)a.s1), dim3(256), 0, st, a);
        hipLaunchKernelGGL(wall_dft_sum, dim3(g1), dim3(256), 0, st, a);
        hipLaunchKernelGGL(wall_synth_part, dim3(g2, (unsigned)std::max(a.s2, 2)), dim3(256), 0, st, a);
        hipLaunchKernelGGL(wall_synth_fin, dim3(grid((int64_t)a.P * a.n_nodes)), dim3(256), 0, st, a);
    }
    return hipGetLastError();
}

hipError_t add_or_write_launch(int64_t n, int accumulate, double *u, double *v, const double *tu, const double *tv,
                               hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(add_or_write, dim3(grid(n)), dim3(256), 0, st, n, accumulate ? 1 : 0, u, v, tu, tv);
    return hipGetLastError();
}

hipError_t fallback_compact_launch(int64_t n, const int32_t *flag, const double *tx, const double *ty, int32_t *list,
                                   int32_t *count, double *cx, double *cy, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fallback_compact, dim3(grid(n)), dim3(256), 0, st, n, flag, tx, ty, list, count, cx, cy);
    return hipGetLastError();
}

hipError_t fallback_scatter_launch(int64_t m, const int32_t *list, const double *t4, double *tu, double *tv,
                                   hipStream_t st) {
    if (m <= 0) return hipSuccess;
    hipLaunchKernelGGL(fallback_scatter, dim3(grid(m)), dim3(256), 0, st, m, list, t4, tu, tv);
    return hipGetLastError();
}

hipError_t zero_int_launch(int32_t *p, int n, hipStream_t st) {
    hipLaunchKernelGGL(zero_int, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n);
    return hipGetLastError();
}

hipError_t delta_combine_launch(int64_t n, int accumulate, double *u, double *v, const double *t, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(delta_combine, dim3(grid(n)), dim3(256), 0, st, n, accumulate ? 1 : 0, u, v, t);
    return hipGetLastError();
}

}  // namespace s2d
