// Single-call pair-sum kernel.  A workgroup of W waves owns one target tile
// (kWave targets) and W consecutive source splits of one split group; its
// waves evaluate pair_sum() (pair_impl.h) on their splits, and wave 0 adds the
// W results in wave order through LDS.  The waves of the first group also sum
// Kress's rule on their targets' own curves (single layer).  With one split
// group (every source in the workgroup) wave 0 then finishes the targets
// itself: the double layer's diagonal limit, the prefactor and the accumulate
// flag, exactly as finalize() does.  With G > 1 groups, or outputs that lie
// over the sources Kress's rule reads, it writes the group's FP64 partial, and
// finalize() adds the G partials in order.
//
// blockIdx -> (tile, group): group = blockIdx % G, tile = blockIdx / G.  The
// dispatcher assigns workgroups to the 8 XCDs round-robin, so with G a
// multiple of 8 each XCD sees only its own groups and streams only their
// sources through its L2; with G = 1 every XCD streams all sources, which
// the planner allows only when the source records fit in one XCD's L2.
#include "pair_impl.h"
#include "self_impl.h"

namespace s2d {

// OWN: Kress's rule too.  Without it the FP32C kernels hold no table of
// logarithms in LDS, and without SHORT no code for short superblocks: a million
// targets at 64 sources, workgroups of a wave, 173 us (228 with both in one
// kernel).
template <int OP, int PREC, int NI, bool OWN, bool SHORT>
// register allocation held to 8 waves per SIMD (64 VGPRs), so that two 16-wave
// workgroups share a CU: every pair kernel fits (the FP64 single layer of three
// images with OWN and SHORT keeps one register in scratch)
__global__ __launch_bounds__(kMaxPairWaves * kWave) __attribute__((amdgpu_waves_per_eu(8, 8)))
void pair_kernel(PairArgs a, FinalArgs f) {
    constexpr bool kTab = OP == S2D_OP_SLP && (PREC == S2D_FP64 || OWN);
    __shared__ __attribute__((aligned(16))) double ltab[kTab ? kLogTabWords : 2];
    __shared__ double red[2][kMaxPairWaves - 1][kWave];
    if constexpr (kTab) fill_log_table(ltab);
    const int lane = threadIdx.x & (kWave - 1);
    // wave index made wave-uniform for the compiler: the split, and with it
    // every source record address, must be uniform so records take the scalar path
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int W = blockDim.x / kWave;
    const int64_t blk = blockIdx.x;
    const int group = (int)(blk % a.n_groups);
    const int64_t tile = blk / a.n_groups;
    double ox[1], oy[1];
    pair_sum<OP, PREC, 1, NI, SHORT>(a, tile, group * W + wid, lane, ltab, ox, oy);
    const int64_t i = tile * kWave + lane;
    if (OWN && group == 0 && i < a.n_trg) {
        double sx, sy;
        kress_self_one(i, f.n_src, f.on_curve, f.on_node, f.curve_off, f.n_curves, f.sx, f.sy, f.nx, f.ny, f.w, f.fx,
                       f.fy, f.kress, ltab, sx, sy, wid, W);
        ox[0] += sx;
        oy[0] += sy;
    }
    if (wid > 0) {
        red[0][wid - 1][lane] = ox[0];
        red[1][wid - 1][lane] = oy[0];
    }
    __syncthreads();
    if (wid != 0) return;
    double sx = ox[0], sy = oy[0];
    for (int w = 1; w < W; ++w) {
        sx += red[0][w - 1][lane];
        sy += red[1][w - 1][lane];
    }
    if (i >= a.n_trg) return;
    if (a.planes) {
        a.part[(int64_t)(2 * group) * a.n_trg + i] = sx;
        a.part[(int64_t)(2 * group + 1) * a.n_trg + i] = sy;
        return;
    }
    final_one(f, i, sx, sy);
}

template <int OP, int PREC, int NI, bool OWN>
static hipError_t launch_t(const Plan &p, const PairArgs &a, const FinalArgs &f, hipStream_t st) {
    if (p.sbs < kSuperBlock)
        hipLaunchKernelGGL((pair_kernel<OP, PREC, NI, OWN, true>), dim3((unsigned)p.n_blocks), dim3(p.waves * kWave), 0,
                           st, a, f);
    else
        hipLaunchKernelGGL((pair_kernel<OP, PREC, NI, OWN, false>), dim3((unsigned)p.n_blocks), dim3(p.waves * kWave), 0,
                           st, a, f);
    return hipGetLastError();
}

template <int PREC, int NI>
static hipError_t launch_ni(const Plan &p, const PairArgs &a, const FinalArgs &f, hipStream_t st) {
    switch (p.op) {
    case S2D_OP_SLP:
        return f.own_rule ? launch_t<S2D_OP_SLP, PREC, NI, true>(p, a, f, st)
                          : launch_t<S2D_OP_SLP, PREC, NI, false>(p, a, f, st);
    case S2D_OP_DLP: return launch_t<S2D_OP_DLP, PREC, NI, false>(p, a, f, st);
    case S2D_OP_SLP_PRESSURE: return launch_t<S2D_OP_SLP_PRESSURE, PREC, NI, false>(p, a, f, st);
    case S2D_OP_DLP_PRESSURE: return launch_t<S2D_OP_DLP_PRESSURE, PREC, NI, false>(p, a, f, st);
    case S2D_OP_SLP_TRACTION: return launch_t<S2D_OP_SLP_TRACTION, PREC, NI, false>(p, a, f, st);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_pair(const Plan &p, const PairArgs &a, const FinalArgs &f, hipStream_t st) {
    if (p.n_blocks <= 0) return hipSuccess;
    if (p.waves < 1 || p.waves > kMaxPairWaves || a.n_groups < 1) return hipErrorInvalidValue;
    // images three at a time when the count allows it
    const int n_img = a.img_hi - a.img_lo + 1;
    const bool f64 = p.mode == S2D_FP64;
    if (n_img % 3 == 0) return f64 ? launch_ni<S2D_FP64, 3>(p, a, f, st) : launch_ni<S2D_FP32C, 3>(p, a, f, st);
    return f64 ? launch_ni<S2D_FP64, 1>(p, a, f, st) : launch_ni<S2D_FP32C, 1>(p, a, f, st);
}

}  // namespace s2d
