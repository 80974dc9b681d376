// The operands of the split products (gemm_split.hip): every float32 element as the exact sum of three bfloat16 pieces, in planes
// [panel of 256 rows][plane][step of 32 k][256 rows][64 bytes], a row's four 16-byte chunks in the places they are read from in LDS.
#pragma once
#include "common.h"

namespace gptq {

constexpr int PSTEPS = SPLIT_K / 32;                  // 32-element steps per plane
constexpr int64_t BLK = 16384;                   // bytes of one (panel, plane, step) block: 256 rows x 64 bytes
constexpr int64_t PANEL_BYTES = 3 * PSTEPS * BLK; // the three planes of one panel of 256 rows

__device__ __forceinline__ uint32_t bf16_rne(float x) {
    const uint32_t u = __float_as_uint(x);
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}
// a = p1 + p2 + p3 (each a bfloat16 bit pattern); the two subtractions are exact
__device__ __forceinline__ void split3(float a, uint32_t& p1, uint32_t& p2, uint32_t& p3) {
    p1 = bf16_rne(a);
    float r = a - __uint_as_float(p1 << 16);
    p2 = bf16_rne(r);
    r -= __uint_as_float(p2 << 16);
    p3 = bf16_rne(r);
}

__device__ __forceinline__ unsigned char* plane_block(unsigned char* planes, int64_t panel, int plane, int step) {
    return planes + ((panel * 3 + plane) * PSTEPS + step) * BLK;
}
// Four consecutive k (the first a multiple of 4) of a row, in all three planes
__device__ __forceinline__ void store_pieces(unsigned char* planes, int64_t row, int k, float4 v) {
    uint32_t p[3][4];
    split3(v.x, p[0][0], p[1][0], p[2][0]);
    split3(v.y, p[0][1], p[1][1], p[2][1]);
    split3(v.z, p[0][2], p[1][2], p[2][2]);
    split3(v.w, p[0][3], p[1][3], p[2][3]);
    const int r = (int)(row & 255), k4 = (k & 31) >> 2;
    const int off = r * 64 + (((k4 >> 1) ^ ((r >> 2) & 3)) << 4) + (k4 & 1) * 8;
#pragma unroll
    for (int pl = 0; pl < 3; ++pl)
        *reinterpret_cast<uint2*>(plane_block(planes, row >> 8, pl, k >> 5) + off) = make_uint2(p[pl][0] | (p[pl][1] << 16), p[pl][2] | (p[pl][3] << 16));
}

}  // namespace gptq
