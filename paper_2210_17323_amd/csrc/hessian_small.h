// Hessian of layers of few channels (hessian_small.hip).
#pragma once
#include "common.h"

namespace gptq {
// Up to how many 16-bit channels these kernels are the faster ones without a workspace.  Measured, us, tiles of 128 / these: 1537 channels 8
// tokens 23.1 / 9.7, 2048 56 / 21, 32768 551 / 223; 2048 13.5 / 12.0, 54 / 32, 547 / 388; 2304 14.2 / 12.9, 57 / 35, 552 / 442; 300 tokens of 2048 19.3 / 18.4;
// 2560 32768 tokens 553 / 598, 3072 624 / 810.  For float32 see hessian_f32_small_tiles (rules.h).
constexpr int64_t SYRK_SMALL_MAX_16 = 2304;
// H[upper] += 2 X X^T, X [n x t] in place: 16-byte aligned rows (ldx a multiple of 16 bytes), any n and t.
int launch_syrk_small(float* H, int64_t ldh, const void* X, int xdtype, int64_t n, int64_t t, int64_t ldx, hipStream_t s);
}  // namespace gptq
