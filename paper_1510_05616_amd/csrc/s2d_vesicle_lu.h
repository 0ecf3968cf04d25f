#pragma once
// LU of the vesicle preconditioner's blocks (vesicle_lu.hip).
#include <hip/hip_runtime.h>

#include <cstdint>

namespace s2d {

constexpr int kTri = 32;         // rows of an inverted diagonal triangle
constexpr int kLuMax = 512;      // largest block, up to two rows per thread

// nc column-major n x n matrices at Pm, factored in place for pc_solve; perm
// [nc][n]: row r of the factors is row perm[r] of the matrix; info [nc]: the
// first zero pivot's index from 1, or 0
hipError_t pc_lu_launch(int n, int nc, double *Pm, int32_t *perm, int32_t *info, hipStream_t st);

}  // namespace s2d
