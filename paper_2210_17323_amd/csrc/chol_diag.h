// The diagonal blocks of the factorisation (chol_diag.hip).
#pragma once
#include "common.h"

namespace gptq {
// The nbk x nbk block at Hblk (16-byte aligned, nbk <= 128; upper triangle read) becomes R, what lies below its diagonal is
// undefined afterwards; dinv receives R^-1 as a dense 128 x 128 block, zeros below the diagonal, the identity past nbk.
// *info: the 1-based column (col_base + column of the block) of the first pivot met that is not positive, unless set before.
int launch_diag_block(float* Hblk, int64_t ld, int nbk, float* dinv, int* info, int col_base, hipStream_t s);
}  // namespace gptq
