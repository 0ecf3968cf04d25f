// The final reduction of a single evaluation (when the pair kernel leaves
// split-group partials, or when there are no sources); the per-target device
// code is in self_impl.h.
#include "self_impl.h"

namespace s2d {

__global__ __launch_bounds__(256) void finalize(FinalArgs a) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.n_trg) return;
    double sx = 0.0, sy = 0.0;
    for (int s = 0; s < a.n_parts; ++s) {
        sx += a.part[(int64_t)(2 * s) * a.n_trg + i];
        sy += a.part[(int64_t)(2 * s + 1) * a.n_trg + i];
    }
    // without sources every on-curve reference is out of range
    if (a.n_parts == 0 && a.own_rule && a.on_curve[i] >= 0) sx = sy = __builtin_nan("");
    final_one(a, i, sx, sy);
}

hipError_t launch_final(const Plan &p, const FinalArgs &a, hipStream_t st) {
    hipLaunchKernelGGL(finalize, dim3((unsigned)((p.n_trg + 255) / 256)), dim3(256), 0, st, a);
    return hipGetLastError();
}

}  // namespace s2d
