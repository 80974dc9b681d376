// What step 3 driven by the Cholesky factor R of H + lambda I needs beside R when the grid is taken per group of 32, 64 or
// 128 columns (Section 4, "Additional Tricks"; Alg. 1).  A group's grid comes from the weights as they stand at its first
// column, so a block is walked on working weights: w + s U_bb with U_bb = R_bb^-1, the inverse of the block's own 128 x 128
// diagonal block (the corrections delta of the block's waiting columns satisfy delta R_bb = s), and inside the block
// Alg. 1 runs on U's diagonal block, which is that same R_bb^-1 because U = R^-1 is block upper triangular.  The product
// s U_bb costs nothing per block: the deferred updates run on Rt = R with every column block scaled by its U_bb, so the
// accumulators hold  sum_i d_i Rt[i][block] = s U_bb  already.
#include "quantize_common.h"

namespace gptq {

// U_bb = R_bb^-1 for every 128 x 128 diagonal block of R, dense with zeros below the diagonal and the identity outside
// a short last block.  One workgroup of 128 threads per block; thread c solves R_bb x = e_c from the bottom up
// (x[i] = (delta_ic - sum_{i<k<=c} R[i][k] x[k]) / R[i][i]), R_bb and the columns in LDS.
__global__ __launch_bounds__(128) void invert_diag_blocks_kernel(const float* R, int64_t ldr, int64_t n, float* Ub) {
    extern __shared__ __align__(16) float inv_sm[];
    float* rs = inv_sm;
    float* xs = inv_sm + QB * (QB + 1);
    const int64_t j0 = (int64_t)blockIdx.x * QB;
    const int c = threadIdx.x;
    for (int q = threadIdx.x; q < QB * QB; q += 128) {
        const int i = q / QB, k = q % QB;
        const int64_t gi = j0 + i, gk = j0 + k;
        rs[i * (QB + 1) + k] = (gi < n && gk < n) ? (k >= i ? R[gi * ldr + gk] : 0.f) : (i == k ? 1.f : 0.f);
    }
    __syncthreads();
    for (int i = QB - 1; i > c; --i) xs[i * (QB + 1) + c] = 0.f;
    for (int i = c; i >= 0; --i) {
        float sum = (i == c) ? 1.f : 0.f;
        for (int k = i + 1; k <= c; ++k) sum = fmaf(-rs[i * (QB + 1) + k], xs[k * (QB + 1) + c], sum);
        xs[i * (QB + 1) + c] = sum / rs[i * (QB + 1) + i];
    }
    __syncthreads();
    float* dst = Ub + (int64_t)blockIdx.x * QB * QB;
    for (int q = threadIdx.x; q < QB * QB; q += 128) dst[q] = xs[(q / QB) * (QB + 1) + (q % QB)];
}

// Rt[rows above the block, block] = R[those rows, block] U_bb, one workgroup per 128 x 128 tile above the diagonal
// blocks (tile number t of the strict upper triangle of blocks, column block by column block).  U_bb sits in LDS, a wavefront makes 16 rows
// on the float32 matrix cores, its operands of them straight from memory: a lane reads 4 consecutive k of a row, and four lanes
// exchange them so that an instruction takes four k in a row, ascending: U_bb's columns end at their largest element, which is added last.
// Bound by these instructions (7 us a tile and CU, 166 of the whole; 3 of the 7 multiply U_bb's zeros, so that what is not finite goes where
// it went) and by a tile's loads ahead of them.  14336 x 14336: 406 us, 912 with a multiply-add per lane and both operands out of LDS.
__global__ __launch_bounds__(512) void scale_column_blocks_kernel(const float* R, int64_t ldr, int64_t n, const float* Ub, float* Rt, int64_t ldt) {
    typedef float floatx4 __attribute__((ext_vector_type(4)));
    int jb = 1, ib = (int)blockIdx.x;                    // tile t -> (ib, jb), ib < jb: column block jb has jb tiles
    while (ib >= jb) { ib -= jb; ++jb; }
    constexpr int P = 144;                    // pitch: the four rows an operand read touches fall on different banks
    extern __shared__ __align__(16) float scale_sm[];
    float* Us = scale_sm;                     // [k][c]
    const int64_t i0 = (int64_t)ib * QB, j0 = (int64_t)jb * QB;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, kq = lane >> 4;
    const float* row = R + (i0 + wave * 16 + l16) * ldr;               // inside the matrix: rows above j0 <= n
    float a[8][4];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const int64_t gk = j0 + 16 * s + 4 * kq;
        if (gk + 4 <= n) {
            const float4 v = *reinterpret_cast<const float4*>(row + gk);
            a[s][0] = v.x; a[s][1] = v.y; a[s][2] = v.z; a[s][3] = v.w;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) a[s][e] = gk + e < n ? row[gk + e] : 0.f;
        }
    }
    // a[s][e] of lane group kq: k = 16 s + 4 kq + e -> 16 s + 4 e + kq
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(a[s][0]), __float_as_uint(a[s][1]), false, false);
        const auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(a[s][2]), __float_as_uint(a[s][3]), false, false);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const auto y = __builtin_amdgcn_permlane32_swap(p[h], q[h], false, false);
            a[s][h] = __uint_as_float(y[0]);
            a[s][h + 2] = __uint_as_float(y[1]);
        }
    }
    const float4* ub = reinterpret_cast<const float4*>(Ub + (int64_t)jb * QB * QB);
#pragma unroll
    for (int i = 0; i < QB * QB / 4 / 512; ++i) {
        const int q = threadIdx.x + 512 * i;
        *reinterpret_cast<float4*>(Us + (q >> 5) * P + (q & 31) * 4) = ub[q];
    }
    __syncthreads();
    floatx4 acc[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) acc[u] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 8; ++s)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int u = 0; u < 8; ++u)
                acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s][e], Us[(16 * s + 4 * e + kq) * P + 16 * u + l16], acc[u], 0, 0, 0);
    // rows 4 kq + i, column 16 u + l16
    float* dst = Rt + (i0 + wave * 16 + 4 * kq) * ldt + j0 + l16;
#pragma unroll
    for (int u = 0; u < 8; ++u)
        if (j0 + 16 * u + l16 < n)
#pragma unroll
            for (int i = 0; i < 4; ++i) dst[i * ldt + 16 * u] = acc[u][i];
}

int launch_invert_diag_blocks(const float* R, int64_t ldr, int64_t n, float* Ub, hipStream_t s) {
    constexpr size_t inv_lds = 2 * QB * (QB + 1) * sizeof(float);
    GPTQ_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(invert_diag_blocks_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)inv_lds));
    hipLaunchKernelGGL(invert_diag_blocks_kernel, dim3((unsigned)ceil_div(n, QB)), dim3(128), inv_lds, s, R, ldr, n, Ub);
    GPTQ_LAUNCH_CHECK();
    return GPTQ_OK;
}

int launch_scale_column_blocks(const float* R, int64_t ldr, int64_t n, const float* Ub, float* Rt, int64_t ldt, hipStream_t s) {
    const int64_t nblk = ceil_div(n, QB);
    if (nblk < 2) return GPTQ_OK;
    if (nblk > 65535) return fail(GPTQ_ERR_UNSUPPORTED, "quantize_layer_from_factor: too many column blocks");
    const int64_t tiles = nblk * (nblk - 1) / 2;
    constexpr size_t lds = QB * 144 * sizeof(float);
    GPTQ_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(scale_column_blocks_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(scale_column_blocks_kernel, dim3((unsigned)tiles), dim3(512), lds, s, R, ldr, n, Ub, Rt, ldt);
    GPTQ_LAUNCH_CHECK();
    return GPTQ_OK;
}

}  // namespace gptq
