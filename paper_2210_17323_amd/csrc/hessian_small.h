// Hessian of layers of few channels (hessian_small.hip).
#pragma once
#include "common.h"

namespace gptq {
// Up to how many 16-bit channels these kernels are the faster ones without a workspace.  Measured, us, tiles of 128 / these: 1540 channels 32
// tokens 20.5 / 11.9, 4096 90 / 34, 32768 550 / 223; 2040 20.1 / 16.7, 87 / 53, 549 / 378; 2300 22.9 / 17.9, 90 / 61, 552 / 440; 2560 8 tokens 15.9 / 19.8, 2048 57 / 48,
// 32768 553 / 598; 3072 20.8 / 26.3, 99 / 105, 624 / 810.  For float32 see hessian_f32_small_tiles (rules.h).
constexpr int64_t SYRK_SMALL_MAX_16 = 2304;
// H[upper] += 2 X X^T, X [n x t] in place: 16-byte aligned rows (ldx a multiple of 16 bytes), any n and t.
int launch_syrk_small(float* H, int64_t ldh, const void* X, int xdtype, int64_t n, int64_t t, int64_t ldx, hipStream_t s);
}  // namespace gptq
