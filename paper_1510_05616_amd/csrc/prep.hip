// Source preparation of a single evaluation (device code in prep_impl.h and
// self_impl.h): records, superblock sums and Kress tables by one launch.  At
// the sizes the direct sum serves each of these is a few microseconds of work,
// less than a launch of its own.
#include "prep_impl.h"
#include "self_impl.h"

namespace s2d {

struct PrepArgs {
    int64_t n_src, n_pad, n_sb;
    int sbs;
    int32_t n_curves;
    int64_t b_rec, b_sum;            // workgroups of records and of superblock sums; then one per curve
    const int32_t *off;
    const double *x, *y, *nx, *ny, *w, *fx, *fy;
    void *rec, *rec64;
    SubInfo *sub;
    double *sbsum, *kress;
};

template <int OP, int PREC>
__global__ __launch_bounds__(256) void prep(PrepArgs a) {
    __shared__ double ctab[OP == S2D_OP_SLP ? kCosTab : 1];
    const int64_t b = blockIdx.x;
    if (b < a.b_rec) {
        const int64_t j = b * 256 + threadIdx.x;
        if (j >= a.n_pad) return;
        if (PREC == S2D_FP64) {
            prep_one64<OP>(j, a.n_src, a.x, a.y, a.nx, a.ny, a.w, a.fx, a.fy, a.rec);
        } else {
            prep_one32<OP>(j, a.n_src, a.x, a.y, a.nx, a.ny, a.w, a.fx, a.fy, a.rec, a.sub);
            // FP64 records for the near sub-blocks of the pressures and traction
            if (a.rec64) prep_one64<OP>(j, a.n_src, a.x, a.y, a.nx, a.ny, a.w, a.fx, a.fy, a.rec64);
        }
    } else if (b < a.b_rec + a.b_sum) {
        const int64_t sb = (b - a.b_rec) * 4 + threadIdx.x / kWave;          // a wave per superblock
        if (sb < a.n_sb)
            sbsum_wave(sb, a.sbs, a.n_src, a.w, a.fx, a.fy, a.sbsum, threadIdx.x & (kWave - 1));
    } else if constexpr (OP == S2D_OP_SLP) {
        kress_table_curve(a.off, (int32_t)(b - a.b_rec - a.b_sum), a.n_src, a.kress, ctab);
    }
}

template <int OP, int PREC>
static hipError_t prep_t(const Plan &p, const s2d_curves *s, void *ws, hipStream_t st) {
    char *b = (char *)ws;
    PrepArgs a{};
    a.n_src = p.n_src;
    a.sbs = p.sbs;
    a.n_sb = p.n_sb;
    a.n_pad = p.n_sb * p.sbs;
    a.off = s->curve_off;
    a.x = s->x;
    a.y = s->y;
    a.nx = s->nx;
    a.ny = s->ny;
    a.w = s->w;
    a.fx = s->fx;
    a.fy = s->fy;
    a.rec = b + p.off_rec;
    a.rec64 = PREC == S2D_FP32C && near_fp64(p.op) ? b + p.off_rec64 : nullptr;
    a.sub = (SubInfo *)(b + p.off_sub);
    a.sbsum = (double *)(b + p.off_sbsum);
    a.kress = (double *)(b + p.off_kress);
    a.b_rec = (a.n_pad + 255) / 256;
    a.b_sum = OP == S2D_OP_SLP && PREC == S2D_FP32C ? (p.n_sb + 3) / 4 : 0;
    const int64_t blocks = a.b_rec + a.b_sum + (p.self ? s->n_curves : 0);
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL((prep<OP, PREC>), dim3((unsigned)blocks), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_prep(const Plan &p, const s2d_curves *s, void *ws, hipStream_t st) {
    const bool f64 = p.mode == S2D_FP64;
    if (p.op == S2D_OP_SLP) return f64 ? prep_t<S2D_OP_SLP, S2D_FP64>(p, s, ws, st) : prep_t<S2D_OP_SLP, S2D_FP32C>(p, s, ws, st);
    if (slp_sources(p.op))       // pressure and traction of the single layer: same records, no log sums
        return f64 ? prep_t<S2D_OP_SLP_PRESSURE, S2D_FP64>(p, s, ws, st)
                   : prep_t<S2D_OP_SLP_PRESSURE, S2D_FP32C>(p, s, ws, st);
    return f64 ? prep_t<S2D_OP_DLP, S2D_FP64>(p, s, ws, st) : prep_t<S2D_OP_DLP, S2D_FP32C>(p, s, ws, st);
}

}  // namespace s2d
