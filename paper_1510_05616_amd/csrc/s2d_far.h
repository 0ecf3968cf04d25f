// Far-field summation (far.hip): large sums of the layers by near
// tiles taken term by term and far clusters through truncated expansions, all
// in FP64.
#pragma once
#include "s2d_internal.h"

namespace s2d {

// Sizes and workspace carve-up of one (sources, targets) pair.
struct FarLayout {
    int64_t ns, nt;            // sources, targets
    int64_t n0, n1, n2, nT;    // source nodes of the three levels, target circles
    int groups;                // near workgroups per target circle
    int64_t nblk;              // sort blocks
    int bits;                  // of a sort key
    size_t key[2], idx[2], hist, base, box, spos, node, tnode, txy, rec, coef, part, kress, self;
    size_t total;
};

FarLayout far_layout(int op, int64_t ns, int64_t nt, bool on_curve);

// Whether the far-field sum is the faster route for these sizes and images;
// reuse: one set-up serves several densities.
bool far_worth(int op, int mode, int64_t ns, int64_t nt, int n_img, bool reuse);

// Whether it is for some operator and number of images: workspaces are sized
// alike for all (the direct sum's cost is highest for four images, counted as
// three ungrouped ones).
bool far_possible(int mode, int64_t ns, int64_t nt);

// Orders sources and targets along a space-filling curve and boxes their
// tiles; with Kress's tables when the single layer's targets sit on curves.
// Depends on the coordinates and curve_off only: one set-up serves any number
// of densities.
hipError_t far_setup(int op, const FarLayout &L, const s2d_curves *src, const s2d_targets *trg, void *ws,
                     hipStream_t st);

// The sum over images img_lo..img_hi for the densities in src, finished and
// written (or added) as `f` says (FinalArgs of the same operator; self and
// part are set here).
// tnx, tny: the targets' normals (traction only).
hipError_t far_sum(int op, const FarLayout &L, const s2d_curves *src, const s2d_targets *trg, const double *tnx,
                   const double *tny, double d, int32_t img_lo, int32_t img_hi, FinalArgs f, void *ws,
                   hipStream_t st);

}  // namespace s2d
