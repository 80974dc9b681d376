// Products of rows with the triangular diagonal block of an outer block of 1024 columns (chol_strip.hip).
#pragma once
#include "common.h"

namespace gptq {
constexpr size_t TRIANGLE_WORDS = (size_t)(8 + 28) * 128 * 128;        // a packed outer block: 2.25 MiB of floats
// Packs the diagonal blocks' inverses (dinv: dense 128 x 128 blocks of the whole matrix) and the tiles above them of outer
// block o of R, for launch_triangle_panel (panel) or launch_triangle_inverse.
int launch_pack_triangle(const float* R, int64_t ld, int64_t n, const float* dinv, int64_t o, bool panel, float* packed, hipStream_t s);
// U_oo = R_oo^-1, [1024 x 1024].  Only the blocks on and right of the diagonal are written (the strictly lower part of a diagonal
// block as zeros).
int launch_triangle_inverse(const float* packed, int64_t n, int64_t o, float* Uoo, hipStream_t s);
// X[rows x columns of outer block o] <- X R_oo^-T, in place; X points at the outer block's first column, ldx % 2 == 0.
int launch_triangle_panel(float* X, int64_t ldx, int64_t rows, const float* packed, int64_t n, int64_t o, hipStream_t s);
// The step of the chain behind diagonal block b (columns j0 .. j0 + nbk - 1): panel[0 : j0 - o0, j0 - o0 ..] = H[o0:j0, b] R_bb^-T
// (panel: 1024 x 1024), H[o0:j0, o0:j0] -= P P^T on the tiles that touch the upper triangle.  launch_copy_panel then puts the
// blocks right of the diagonal blocks from `panel` into H, whose outer block is ow columns wide.
int launch_chol_step(float* H, int64_t ld, int64_t o0, int64_t j0, int nbk, const float* dinv_b, float* panel, hipStream_t s);
int launch_copy_panel(float* H, int64_t ld, int64_t o0, int ow, const float* panel, hipStream_t s);
}  // namespace gptq
