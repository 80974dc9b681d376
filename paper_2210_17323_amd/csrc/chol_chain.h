// The serial chain of the factorisation inside one outer block of 1024 columns (chol_chain.hip).
#pragma once
#include "common.h"

namespace gptq {
constexpr size_t CHAIN_FLAG_BYTES = 256;
constexpr int CHAIN_TIMED_OUT = -1;      // in *info: workgroups that wait for one another gave up
// The outer block at columns o0 .. o0 + ow - 1 of H (16-byte aligned, ld % 4 == 0; upper triangle read) becomes R, what lies below
// the diagonal of its diagonal blocks is undefined afterwards; dinv receives R_bb^-1 of its blocks as dense 128 x 128 blocks,
// zeros below the diagonal, the identity past ow.  panel: 1024 x 1024 floats of scratch, 256-byte aligned.  packed (null: not
// wanted): the outer block as launch_triangle_panel reads it.  flags: CHAIN_FLAG_BYTES that hold zeros or what launches of smaller epochs
// (> 0) left.  *info: the 1-based column (o0 + column) of a pivot that is not positive, or CHAIN_TIMED_OUT, unless set before.
int launch_chol_chain(float* H, int64_t ld, int64_t o0, int ow, float* dinv, float* panel, float* packed, int* flags, int epoch, int* info, hipStream_t s);
}  // namespace gptq
