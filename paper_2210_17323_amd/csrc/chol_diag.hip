// The serial part of step 2 (Section 3, Step 3): one 128 x 128 diagonal block D = R R^T, R upper triangular, taken from the
// last column backwards, and R^-1.
//
// With rows and columns numbered from the last one, i' = 127 - i, this is the ordinary Cholesky factorisation L L^T, and
// R^-1 is L^-1; everything below is in that numbering.  Panels of 16 columns, p = 0 .. 7:
//   panel   A 16 x 16 diagonal block is factored by the 16 lanes of a DPP row, a row per lane, in registers: column j of the
//           block, needed by every lane, is register j, read from lane k of the own DPP row inside the multiply-add.
//           Every DPP row of a wavefront does this with its own copy of the block while its lanes solve another 16 rows
//           of the panel with the same broadcasts, so the panel below costs no more than the block.  The lanes whose
//           rows are the diagonal block itself solve the identity, which gives L_pp^-1.
//   chol    The rest of the matrix, 16 x 16 tiles as accumulators of v_mfma_f32_16x16x4_f32 spread over 8 wavefronts,
//           loses the panel's products;
//   inverse X_pc = L_pp^-1 X_pc, then X_ic -= L_ip X_pc for the rows below, X = L^-1 in accumulators too.
// Three barriers a panel.  What bounds it is the chain of 128 pivots, ~150 cycles each, then latency of 8 x 3 barriers and of the
// load.  Measured: 28 us a block with the chip to itself, 36 us on the mean beside the trailing updates of a 12288 x 12288
// matrix; 37 us alone when the blocks were 32 x 32 with their columns handed round through LDS.
#include "chol_diag.h"

#include <utility>

namespace gptq {

typedef float floatx4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int DB = 128, PB = 16, NP = DB / PB;
constexpr int PP = 20;                  // pitch of the panel in LDS (16-byte aligned rows on different banks)
constexpr int XP = 132;                 // pitch of a row block of X
constexpr int WAVES = 8;
constexpr int CT = (NP * (NP + 1) / 2 + WAVES - 1) / WAVES;      // matrix tiles per wavefront: 5
constexpr int XT = (NP * (NP - 1) / 2 + WAVES - 1) / WAVES;      // tiles of X strictly below the diagonal: 4

// tile number -> (i, c), i >= c, of the lower triangle with its diagonal
__device__ __forceinline__ void tile_of(int t, int& i, int& c) { i = 0; while (t > i) { t -= i + 1; ++i; } c = t; }

// w -= m * (u of lane C of the own DPP row)
template <int C>
__device__ __forceinline__ void fma_bcast16(float& w, float u, float m) {
    asm volatile("v_fmac_f32_dpp %0, %1, -%2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(w) : "v"(u), "v"(m), "n"(C));
}

template <int J, int... K>
__device__ __forceinline__ void update_right(float (&dx)[PB], float (&px)[PB], float col, float du, float pu, std::integer_sequence<int, K...>) {
    // columns J + 1 + K: the next pivot's column first
    ((fma_bcast16<J + 1 + K>(dx[J + 1 + K], col, du), fma_bcast16<J + 1 + K>(px[J + 1 + K], col, pu)), ...);
}

// Pivot J: dx[J] and px[J] become the column of L.  The update multiplies the column as it stands with the row's entry over the
// pivot, so that an element loses one product with two roundings; 1 / sqrt(pivot) is the hardware's estimate with one Newton
// step whose residual 1 - pivot * inv^2 is taken without the rounding of pivot * inv (half an ulp in all: the first digit
// the whole factorisation loses).  `mine` keeps the pivot of this lane's row.
template <int J>
__device__ __forceinline__ void pivot(float (&dx)[PB], float (&px)[PB], float& mine, int l16) {
    asm volatile("s_nop 1" : "+v"(dx[J]));              // last written by a statement the compiler cannot see into
    const float dd = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, dx[J]), 0x150 + J, 0xf, 0xf, true));     // row_newbcast
    const float est = __builtin_amdgcn_rsqf(dd);
    const float t = dd * est;
    const float e = fmaf(-fmaf(dd, est, -t), est, fmaf(-t, est, 1.f));
    const float inv = fmaf(0.5f * est, e, est);
    mine = l16 == J ? dd : mine;
    float col = dx[J];
    dx[J] *= inv;
    px[J] *= inv;
    if constexpr (J + 1 < PB) {
        const float du = dx[J] * inv, pu = px[J] * inv;
        asm volatile("s_nop 1" : "+v"(col));            // the wait states between a vector write and a DPP read
        update_right<J>(dx, px, col, du, pu, std::make_integer_sequence<int, PB - 1 - J>{});
    }
}

template <int... J>
__device__ __forceinline__ void pivots(float (&dx)[PB], float (&px)[PB], float& mine, int l16, std::integer_sequence<int, J...>) {
    (pivot<J>(dx, px, mine, l16), ...);
}

__device__ __forceinline__ void barrier_lds() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

}  // namespace

__global__ __launch_bounds__(64 * WAVES) void diag_block_kernel(float* Hblk, int64_t ld, int nbk, float* dinv, int* info, int col_base) {
    __shared__ __attribute__((aligned(16))) float panel[2][DB * PP];       // columns 16 p .. of rows 16 p ..: before, then L
    __shared__ __attribute__((aligned(16))) float xrow[2][PB * XP];        // row block p of X
    __shared__ __attribute__((aligned(16))) float linv_t[PB * PP];         // (L_pp^-1)^T
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, kq = lane >> 4;

    floatx4 ch[CT], xt[XT];
    int ci[CT], cc[CT], xi[XT], xc[XT];
#pragma unroll
    for (int s = 0; s < CT; ++s) {
        const int t = wave + WAVES * s;
        ci[s] = cc[s] = -1;
        if (t < NP * (NP + 1) / 2) tile_of(t, ci[s], cc[s]);
        ch[s] = floatx4{0.f, 0.f, 0.f, 0.f};
        if (ci[s] < 0) continue;
#pragma unroll
        for (int e = 0; e < 4; ++e) {                    // element (16 i + 4 kq + e, 16 c + l16) of the reversed block
            const int a = DB - 1 - (PB * ci[s] + 4 * kq + e), b = DB - 1 - (PB * cc[s] + l16);
            ch[s][e] = (a < nbk && b < nbk) ? Hblk[(int64_t)min(a, nbk - 1) * ld + min(b, nbk - 1)] : (a == b ? 1.f : 0.f);
        }
    }
#pragma unroll
    for (int s = 0; s < XT; ++s) {
        const int t = wave + WAVES * s;
        xi[s] = xc[s] = -1;
        if (t < NP * (NP - 1) / 2) { tile_of(t, xi[s], xc[s]); ++xi[s]; }        // strictly below: (i + 1, c)
        xt[s] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    int bad_col = -1;
    // tiles of column p (and the row block p of X) to LDS
    auto extract = [&](int p) {
#pragma unroll
        for (int s = 0; s < CT; ++s)
            if (cc[s] == p) {
#pragma unroll
                for (int e = 0; e < 4; ++e) panel[p & 1][(PB * ci[s] + 4 * kq + e) * PP + l16] = ch[s][e];
            }
#pragma unroll
        for (int s = 0; s < XT; ++s)
            if (xi[s] == p) {
#pragma unroll
                for (int e = 0; e < 4; ++e) xrow[p & 1][(4 * kq + e) * XP + PB * xc[s] + l16] = xt[s][e];
            }
    };
    extract(0);
    barrier_lds();
#pragma unroll 1
    for (int p = 0; p < NP; ++p) {
        float* pn = panel[p & 1];
        float* xr = xrow[p & 1];
        if (wave < 2 && 64 * wave + 63 >= PB * p) {
            const int row = 64 * wave + lane;            // the row of the panel this lane solves
            const bool own = (row >> 4) == p;            // ... the diagonal block's: the identity instead
            float dx[PB], px[PB];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const floatx4 d = *reinterpret_cast<const floatx4*>(&pn[(PB * p + l16) * PP + 4 * q]);
                const floatx4 x = *reinterpret_cast<const floatx4*>(&pn[max(row, PB * p) * PP + 4 * q]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    dx[4 * q + e] = d[e];
                    px[4 * q + e] = own ? (l16 == 4 * q + e ? 1.f : 0.f) : x[e];
                }
            }
            float mine = 0.f;
            pivots(dx, px, mine, l16, std::make_integer_sequence<int, PB>{});
            {
                const uint32_t bad = (uint32_t)__ballot(!(mine > 0.f)) & 0xffffu;
                if (bad && bad_col < 0) bad_col = PB * p + __builtin_ctz(bad);
            }
            const float root = __fsqrt_rn(mine);         // the diagonal of L
            if (row >= PB * p) {
                // R: row 127 - row, columns 127 - 16 p - 15 .. 127 - 16 p
                const int a = DB - 1 - row, b0 = DB - 1 - PB * p - 15;
                float v[PB];
#pragma unroll
                for (int k = 0; k < PB; ++k) v[k] = own ? (k < l16 ? dx[k] : (k == l16 ? root : 0.f)) : px[k];
                if (a < nbk) {
                    float* dst = Hblk + (int64_t)a * ld + b0;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        if (b0 + 4 * q + 4 <= nbk) *reinterpret_cast<floatx4*>(dst + 4 * q) = floatx4{v[15 - 4 * q], v[14 - 4 * q], v[13 - 4 * q], v[12 - 4 * q]};
                        else {
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                if (b0 + 4 * q + e < nbk) dst[4 * q + e] = v[15 - 4 * q - e];
                        }
                    }
                }
                if (own) {
#pragma unroll
                    for (int k = 0; k < PB; ++k) xr[k * XP + PB * p + l16] = px[k];           // X_pp[k][l16]
#pragma unroll
                    for (int q = 0; q < 4; ++q) *reinterpret_cast<floatx4*>(&linv_t[l16 * PP + 4 * q]) = floatx4{px[4 * q], px[4 * q + 1], px[4 * q + 2], px[4 * q + 3]};
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q) *reinterpret_cast<floatx4*>(&pn[row * PP + 4 * q]) = floatx4{px[4 * q], px[4 * q + 1], px[4 * q + 2], px[4 * q + 3]};
                }
            }
        }
        barrier_lds();
        // the matrix tiles right of the panel, and this row block of X
#pragma unroll
        for (int s = 0; s < CT; ++s)
            if (cc[s] > p) {
                const floatx4 a = *reinterpret_cast<const floatx4*>(&pn[(PB * ci[s] + l16) * PP + 4 * kq]);
                const floatx4 b = *reinterpret_cast<const floatx4*>(&pn[(PB * cc[s] + l16) * PP + 4 * kq]);
                floatx4 v = {0.f, 0.f, 0.f, 0.f};        // the panel's 16 products, subtracted at once: one by one, each would
#pragma unroll
                for (int e = 0; e < 4; ++e) v = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], v, 0, 0, 0);      // be rounded at the size of the element
                ch[s] -= v;
            }
        if (wave < p) {
            floatx4 x = {0.f, 0.f, 0.f, 0.f};            // X_p,wave = L_pp^-1 X_p,wave, in place
#pragma unroll
            for (int e = 0; e < 4; ++e)
                x = __builtin_amdgcn_mfma_f32_16x16x4f32(linv_t[(4 * kq + e) * PP + l16], xr[(4 * kq + e) * XP + PB * wave + l16], x, 0, 0, 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) xr[(4 * kq + e) * XP + PB * wave + l16] = x[e];
        }
        barrier_lds();
        // the rows of X below, and row block p of X = rows 127 - 16 p - 15 .. of R^-1 to memory
#pragma unroll
        for (int s = 0; s < XT; ++s)
            if (xi[s] > p && xc[s] <= p) {
                const floatx4 a = *reinterpret_cast<const floatx4*>(&pn[(PB * xi[s] + l16) * PP + 4 * kq]);
                floatx4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int e = 0; e < 4; ++e) v = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], xr[(4 * kq + e) * XP + PB * xc[s] + l16], v, 0, 0, 0);
                xt[s] -= v;
            }
        {
            const int m = tid >> 5, b = (tid & 31) * 4;  // row of the block, first of four columns of R^-1
            const int k = DB - 1 - b;                    // ... which is this one of X, descending
            floatx4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (k - e) < PB * (p + 1) ? xr[m * XP + k - e] : 0.f;
            *reinterpret_cast<floatx4*>(dinv + (DB - 1 - PB * p - m) * DB + b) = v;
        }
        if (p + 1 < NP) extract(p + 1);
        barrier_lds();
    }
    if (bad_col >= 0 && lane == 0) atomicCAS(info, 0, col_base + DB - bad_col);     // column 127 - bad_col, counted from 1
}

int launch_diag_block(float* Hblk, int64_t ld, int nbk, float* dinv, int* info, int col_base, hipStream_t s) {
    hipLaunchKernelGGL(diag_block_kernel, dim3(1), dim3(64 * WAVES), 0, s, Hblk, ld, nbk, dinv, info, col_base);
    GPTQ_LAUNCH_CHECK();
    return GPTQ_OK;
}

}  // namespace gptq
