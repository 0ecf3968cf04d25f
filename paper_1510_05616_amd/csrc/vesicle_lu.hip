// Factorisation of the vesicle preconditioner's blocks: LU with partial
// pivoting of nc dense n x n matrices (column-major, n up to kLuMax), one
// workgroup each, in the form pc_solve (vesicle.hip) reads: rows permuted,
// L strictly below and U on and above the diagonal, each kTri x kTri diagonal
// block's triangles replaced by their inverses, and the permutation.
//
// Panels of kTri columns.  A thread holds its row of the panel in registers
// (rows past the workgroup's threads are in LDS); a column's pivot has the
// largest high word (20 bits of mantissa, the first row of equals), so it is
// within 1e-6 of the largest.  It is found by DPP within a wave; each wave
// offers its best row in LDS and all take the best offer: one barrier a column.
// Rows are relabelled, not moved.  One wave inverts the diagonal block's
// triangles; U12 = L11^-1 A12 and the trailing update are 16 x 16 x 4 FP64
// matrix products that read their rows through the relabelling; columns left of
// the panel are permuted once at the end.
//
// 1,000 blocks of 288 (0.66 MB each): 1.95 ms, against 3.1 ms for the library's
// batched factorisation and 0.66 ms for the inversions after it; 32 blocks 0.62
// ms.  Bound by the chain of a column step (about 2,000 cycles) for few blocks
// and for many by the trailing update's passes over blocks that only the last
// cache holds: two workgroups per CU (256 registers) are as fast as four with
// 128 registers, and sharing L's loads among more columns changed nothing.
#include "self_impl.h"
#include "s2d_vesicle_lu.h"

#include <algorithm>
#include <utility>

namespace s2d {

namespace {

constexpr int kThreads = 256, kWaves = kThreads / kWave;
using d4 = double __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t wave_umax(uint32_t x) {
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x121, 0xf, 0xf, false));   // row_ror:1
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x122, 0xf, 0xf, false));
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x124, 0xf, 0xf, false));
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xf, 0xf, false));
    const uint32_t a = max((uint32_t)__builtin_amdgcn_readlane((int)x, 0), (uint32_t)__builtin_amdgcn_readlane((int)x, 16));
    const uint32_t b = max((uint32_t)__builtin_amdgcn_readlane((int)x, 32), (uint32_t)__builtin_amdgcn_readlane((int)x, 48));
    return max(a, b);
}

// a wave's pivot candidate: high word of its magnitude plus 1 (0: none), row
// of the panel, position, and the row's values
struct alignas(16) Offer {
    uint32_t key;
    int row, pos, pad;
    double v[kTri];
};

// f(0), f(1), .. f(N - 1) with constant arguments: register arrays indexed by
// them stay in registers where the unroller leaves a loop with barriers alone
template <class F, int... I>
__device__ __forceinline__ void unrolled_seq(F &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void unrolled(F &&f) { unrolled_seq(f, std::make_integer_sequence<int, N>{}); }

__device__ __forceinline__ uint32_t key_of(double v, bool done) {
    return done ? 0u : ((uint32_t)__double2hiint(v) & 0x7fffffffu) + 1u;
}

// v / piv from ip, 1 / piv to one step: exact where the quotient is a double,
// so that rows equal up to a factor cancel to an exact zero pivot
__device__ __forceinline__ double quotient(double v, double piv, double ip) {
    const double q = v * ip;
    return __builtin_fma(__builtin_fma(-q, piv, v), ip, q);
}

// dynamic LDS: rows kThreads.. of a panel, column by column, then the 16-bit
// tables src and fin [n] and snap [panels][n]
size_t lu_lds(int n) {
    const int ne = std::max(n - kThreads, 0), np = (n + kTri - 1) / kTri;
    return (size_t)ne * kTri * sizeof(double) + (size_t)(np + 2) * n * sizeof(uint16_t);
}

__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void pc_lu(int n, double *Pm, int32_t *perm, int32_t *info) {
    // [0] the diagonal block, [1] the same read backwards, both column by column;
    // then the inverses of L and (rows backwards) of U
    constexpr int kLd = kTri + 2;
    __shared__ __attribute__((aligned(16))) double tile[2][kTri][kLd];
    __shared__ Offer offer[2][kWaves];              // by parity of the column: one barrier each
    extern __shared__ double dyn[];
    const int ne = max(n - kThreads, 0);
    double *ext = dyn;                              // [kTri][ne]
    uint16_t *src = (uint16_t *)(dyn + ne * kTri);  // position -> position before the panel
    uint16_t *fin = src + n;                        // row -> final position
    uint16_t *snap = fin + n;                       // [panel][position] -> row, after the panel
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wid = __builtin_amdgcn_readfirstlane(tid / kWave), lo16 = lane & 15, hi4 = lane >> 4;
    double *A = Pm + (int64_t)blockIdx.x * n * n;
    // element (r, c), by a 32-bit offset from the workgroup's base
    const auto el = [&](uint32_t r, uint32_t c) -> double & {
        return *(double *)((char *)A + (size_t)(8u * (r + c * (uint32_t)n)));
    };
    int sing = 0, p = 0;
    for (int k0 = 0; k0 < n; k0 += kTri, ++p) {
        const int nb = min(kTri, n - k0);
        const bool two = n - k0 > kThreads;         // rows k0 + kThreads.. in ext
        const bool live = k0 + tid < n, live2 = k0 + kThreads + tid < n;
        double v[kTri];
#pragma unroll
        for (int c = 0; c < kTri; ++c) v[c] = live && c < nb ? el(k0 + tid, k0 + c) : 0.0;
        if (two && live2)
            for (int c = 0; c < kTri; ++c) ext[c * ne + tid] = c < nb ? el(k0 + kThreads + tid, k0 + c) : 0.0;
        int pos = k0 + tid, pos2 = pos + kThreads;
        bool done = !live, done2 = !live2;
        unrolled<kTri>([&](auto J) {
            constexpr int j = decltype(J)::value;
            if (j >= nb) return;
            uint32_t key = key_of(v[j], done);
            bool second = false;
            if (two) {
                const uint32_t k2 = key_of(live2 ? ext[j * ne + tid] : 0.0, done2);
                second = k2 > key;
                key = max(key, k2);
            }
            const uint32_t m = wave_umax(key);
            // each wave offers its best row; the best offer of all is the pivot
            Offer &o = offer[j & 1][wid];
            if (lane == __builtin_ctzll(__ballot(key == m))) {
                o.key = m;
                o.row = second ? tid + kThreads : tid;
                o.pos = second ? pos2 : pos;
                if (!second) {
#pragma unroll
                    for (int c = j; c < kTri; ++c) o.v[c] = v[c];
                } else {
#pragma unroll 4
                    for (int c = j; c < kTri; ++c) o.v[c] = ext[c * ne + tid];
                }
            }
            __syncthreads();
            const uint32_t k = offer[j & 1][lane & (kWaves - 1)].key;
            const int win = __builtin_ctzll(__ballot(k == wave_umax(k)));
            const Offer &b = offer[j & 1][win];
            const int who = b.row, from = b.pos;
            const double piv = b.v[j], ip = rcp64(piv);
            const auto relabel = [&](int r, int &q, bool &d) {
                if (r == who) {
                    q = k0 + j;
                    d = true;
                } else if (q == k0 + j) {
                    q = from;
                }
            };
            if (live) relabel(tid, pos, done);
            if (piv == 0.0 && sing == 0) sing = k0 + j + 1;
            if (!done) {
                const double l = quotient(v[j], piv, ip);
                v[j] = l;
#pragma unroll
                for (int c = j + 1; c < kTri; ++c) v[c] = __builtin_fma(-l, b.v[c], v[c]);
            }
            if (two && live2) {
                relabel(tid + kThreads, pos2, done2);
                if (!done2) {
                    const double l = quotient(ext[j * ne + tid], piv, ip);
                    ext[j * ne + tid] = l;
#pragma unroll 4
                    for (int c = j + 1; c < kTri; ++c)
                        ext[c * ne + tid] = __builtin_fma(-l, b.v[c], ext[c * ne + tid]);
                }
            }
        });
        // the panel's rows to their places; a row's identity is that of the
        // position it came from
        const auto place = [&](int from, int q, auto &&val) {
            src[q] = (uint16_t)from;
            snap[p * n + q] = p ? snap[(p - 1) * n + from] : (uint16_t)from;
            if (q < k0 + kTri) {
#pragma unroll
                for (int c = 0; c < kTri; ++c) {
                    tile[0][c][q - k0] = val(c);
                    tile[1][kTri - 1 - c][kTri - 1 - (q - k0)] = val(c);
                }
            } else {
#pragma unroll
                for (int c = 0; c < kTri; ++c)
                    if (c < nb) el(q, k0 + c) = val(c);
            }
        };
        if (live) place(k0 + tid, pos, [&](int c) { return v[c]; });
        if (two && live2) place(k0 + kThreads + tid, pos2, [&](int c) { return ext[c * ne + tid]; });
        for (int q = tid; q < k0; q += kThreads) snap[p * n + q] = snap[(p - 1) * n + q];
        // a short last block is completed by the identity
        for (int e = tid; e < (kTri - nb) * kTri; e += kThreads) {
            const int r = nb + e / kTri, c = e % kTri;
            tile[0][c][r] = tile[1][kTri - 1 - c][kTri - 1 - r] = r == c ? 1.0 : 0.0;
        }
        __syncthreads();
        if (wid == 0) {
            // lane c: column c of L11^-1, lane 32 + c: column c of U11^-1,
            // whose triangle is read backwards to make the same substitution
            const bool up = lane >= kTri;
            const int c = lane & (kTri - 1), ci = up ? kTri - 1 - c : c;
            const double *t = &tile[up][0][0];
            tile[up][c][c] = up ? 1.0 / tile[1][c][c] : 1.0;     // the diagonals' inverses first
            double x[kTri];
#pragma unroll
            for (int r = 0; r < kTri; ++r) x[r] = r == ci ? 1.0 : 0.0;
#pragma unroll
            for (int k = 0; k < kTri; ++k) {
                asm volatile("" ::: "memory");      // a column's loads at a time
                x[k] *= t[k * kLd + k];
#pragma unroll
                for (int r = k + 1; r < kTri; ++r) {
                    if (r % 16 == 0) asm volatile("" ::: "memory");
                    x[r] = __builtin_fma(-t[k * kLd + r], x[k], x[r]);
                }
            }
            double *o = &tile[up][c][0];
#pragma unroll
            for (int r = 0; r < kTri; ++r) o[r] = x[r];
        }
        __syncthreads();
        for (int e = tid; e < nb * kTri; e += kThreads) {
            const int i = e % kTri, c = e / kTri;
            if (i < nb) el(k0 + i, k0 + c) = i > c ? tile[0][c][i] : tile[1][c][kTri - 1 - i];
        }
        // trailing columns, 16 at a time by wave (nb = kTri where there are any)
        for (int c0 = k0 + kTri + 16 * wid; c0 < n; c0 += 16 * kWaves) {
            const bool cok = c0 + lo16 < n;
            double b[8];
#pragma unroll
            for (int s = 0; s < 8; ++s) b[s] = cok ? el(src[k0 + 4 * s + hi4], c0 + lo16) : 0.0;
            // U12: register r of half h holds row 16 h + 4 r + hi4, column lo16
            d4 u[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int s = 0; s < 8; ++s)
                    u[h] = __builtin_amdgcn_mfma_f64_16x16x4f64(tile[0][4 * s + hi4][16 * h + lo16], b[s], u[h], 0, 0, 0);
            // transposed trailing tiles: rows across lanes, columns 4 r + hi4 in
            // register r; u's layout is the left operand's
            for (int r0 = k0 + kTri; r0 < n; r0 += 16) {
                const int rw = r0 + lo16;
                const bool rok = rw < n;
                const int from = rok ? src[rw] : 0;
                d4 t;
                double l[8];
#pragma unroll
                for (int r = 0; r < 4; ++r) t[r] = rok && c0 + 4 * r + hi4 < n ? el(from, c0 + 4 * r + hi4) : 0.0;
#pragma unroll
                for (int s = 0; s < 8; ++s) l[s] = rok ? el(rw, k0 + 4 * s + hi4) : 0.0;
#pragma unroll
                for (int s = 0; s < 8; ++s)
                    t = __builtin_amdgcn_mfma_f64_16x16x4f64(-u[s / 4][s % 4], l[s], t, 0, 0, 0);
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (rok && c0 + 4 * r + hi4 < n) el(rw, c0 + 4 * r + hi4) = t[r];
            }
            // U12 last: rows displaced by the pivots were read from its place
            if (cok) {
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int r = 0; r < 4; ++r) el(k0 + 16 * h + 4 * r + hi4, c0 + lo16) = u[h][r];
            }
        }
        __syncthreads();
    }
    // the panels' rows below their diagonal blocks follow the later pivots
    const uint16_t *last = snap + (p - 1) * n;
    for (int i = tid; i < n; i += kThreads) {
        fin[last[i]] = (uint16_t)i;
        perm[(int64_t)blockIdx.x * n + i] = last[i];
    }
    if (tid == 0) info[blockIdx.x] = sing;
    __syncthreads();
    for (int q = 0, k0 = 0; k0 + kTri < n; ++q, k0 += kTri) {
        constexpr int kHalf = kTri / 2, kRows = kLuMax / kThreads;
        int to[kRows];
#pragma unroll
        for (int e = 0; e < kRows; ++e) {
            const int i = tid + e * kThreads;
            to[e] = i >= k0 + kTri && i < n ? fin[snap[q * n + i]] : i;
        }
        for (int c0 = k0; c0 < k0 + kTri; c0 += kHalf) {
            double v[kRows][kHalf];
#pragma unroll
            for (int e = 0; e < kRows; ++e)
                if (to[e] != tid + e * kThreads) {
#pragma unroll
                    for (int c = 0; c < kHalf; ++c) v[e][c] = el(tid + e * kThreads, c0 + c);
                }
            __syncthreads();
#pragma unroll
            for (int e = 0; e < kRows; ++e)
                if (to[e] != tid + e * kThreads) {
#pragma unroll
                    for (int c = 0; c < kHalf; ++c) el(to[e], c0 + c) = v[e][c];
                }
        }
    }
}

}  // namespace

hipError_t pc_lu_launch(int n, int nc, double *Pm, int32_t *perm, int32_t *info, hipStream_t st) {
    if (n < 1 || n > kLuMax) return hipErrorInvalidValue;
    if (nc <= 0) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute((const void *)pc_lu, hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)lu_lds(kLuMax));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(pc_lu, dim3((unsigned)nc), dim3(kThreads), lu_lds(n), st, n, Pm, perm, info);
    return hipGetLastError();
}

}  // namespace s2d
