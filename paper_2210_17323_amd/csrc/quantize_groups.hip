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
// blocks (tile number t of the strict upper triangle of blocks, column block by column block).  Both operands sit in
// LDS; a thread makes 8 x 4 outputs: its 8 values of a column of A are the same for the 32 threads that share its
// rows (broadcast reads), its 4 values of a row of U_bb one 16-byte read.
__global__ __launch_bounds__(512) void scale_column_blocks_kernel(const float* R, int64_t ldr, int64_t n, const float* Ub, float* Rt, int64_t ldt) {
    int jb = 1, ib = (int)blockIdx.x;                    // tile t -> (ib, jb), ib < jb: column block jb has jb tiles
    while (ib >= jb) { ib -= jb; ++jb; }
    extern __shared__ __align__(16) float scale_sm[];
    constexpr int PA = 133, P = 132;          // pitches: the rows a wavefront reads of A at a time fall on different banks
    float* As = scale_sm;                     // [i][k]
    float* Us = scale_sm + QB * PA;           // [k][c]; 128 * 133 floats is a multiple of 16 bytes
    const int64_t i0 = (int64_t)ib * QB, j0 = (int64_t)jb * QB;
    const float* ub = Ub + (int64_t)jb * QB * QB;
    for (int q = threadIdx.x; q < QB * QB; q += 512) {
        const int i = q / QB, k = q % QB;
        const int64_t gk = j0 + k;
        As[i * PA + k] = (gk < n) ? R[(i0 + i) * ldr + gk] : 0.f;       // rows i0 + i < j0 <= n are inside the matrix
        Us[i * P + k] = ub[q];                                         // row i of U_bb, column k
    }
    __syncthreads();
    const int ty = threadIdx.x >> 5, tx = threadIdx.x & 31;            // rows ty*8 .. +7, columns tx*4 .. +3
    float acc[8][4];
#pragma unroll
    for (int a = 0; a < 8; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = 0.f;
#pragma unroll 4
    for (int k = 0; k < QB; ++k) {
        float av[8];
#pragma unroll
        for (int a = 0; a < 8; ++a) av[a] = As[(ty * 8 + a) * PA + k];
        const float4 b0 = *reinterpret_cast<const float4*>(Us + k * P + tx * 4);
        const float bv[4] = {b0.x, b0.y, b0.z, b0.w};
#pragma unroll
        for (int a = 0; a < 8; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[a][b] = fmaf(av[a], bv[b], acc[a][b]);
    }
#pragma unroll
    for (int a = 0; a < 8; ++a) {
        float* dst = Rt + (i0 + ty * 8 + a) * ldt + j0 + tx * 4;
        if (j0 + tx * 4 + 4 <= n) {
            *reinterpret_cast<float4*>(dst) = make_float4(acc[a][0], acc[a][1], acc[a][2], acc[a][3]);
        } else {
#pragma unroll
            for (int b = 0; b < 4; ++b)
                if (j0 + tx * 4 + b < n) dst[b] = acc[a][b];
        }
    }
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
    constexpr size_t lds = (QB * 133 + QB * 132) * sizeof(float);
    GPTQ_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(scale_column_blocks_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(scale_column_blocks_kernel, dim3((unsigned)tiles), dim3(512), lds, s, R, ldr, n, Ub, Rt, ldt);
    GPTQ_LAUNCH_CHECK();
    return GPTQ_OK;
}

}  // namespace gptq
