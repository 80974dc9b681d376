// Hessian of layers of few channels (hessian_small.hip).
#pragma once
#include "common.h"

namespace gptq {
// Up to how many 16-bit channels these kernels are the faster ones without a workspace: at 2000 the larger tiles are ahead (1.17 ms
// against 1.22 for 65536 tokens).  For float32 see hessian_f32_small_tiles (rules.h).
constexpr int64_t SYRK_SMALL_MAX_16 = 1536;
// H[upper] += 2 X X^T, X [n x t] in place: 16-byte aligned rows (ldx a multiple of 16 bytes), any n and t.
int launch_syrk_small(float* H, int64_t ldh, const void* X, int xdtype, int64_t n, int64_t t, int64_t ldx, hipStream_t s);
}  // namespace gptq
