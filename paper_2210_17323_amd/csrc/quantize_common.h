// Shared by the translation units of step 3 (Algorithm 1): the conversion helpers, the grid of Section 4 from a range of weights,
// and the interface of the strip kernel that walks the columns of one outer block.
#pragma once
#include "common.h"
#include "rules.h"

namespace gptq {

// ---- W (f16 / bf16 / f32) -> float32 working copy; optionally the per-row grid from the original row.
template <typename T> __device__ __forceinline__ float to_f32(T v);
template <> __device__ __forceinline__ float to_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ float to_f32<_Float16>(_Float16 v) { return (float)v; }
template <> __device__ __forceinline__ float to_f32<__bf16>(__bf16 v) { return (float)v; }

__device__ __forceinline__ void grid_from_range(int grid, float maxq, float lo, float hi, float amax, float& scale, int& zero) {
    if (grid == GPTQ_GRID_TERNARY) {
        scale = (amax == 0.f) ? 1.f : amax;
        zero = 1;
    } else {
        lo = fminf(lo, 0.f);
        hi = fmaxf(hi, 0.f);
        if (hi == lo) { scale = 1.f; zero = 0; }
        else {
            scale = (hi - lo) / maxq;
            zero = (int)rintf(-lo / scale);
        }
    }
}

// ---- the walk of one outer block (quantize_strip.hip) ----
constexpr size_t STRIP_DIAG_BYTES = 38912;             // a packed diagonal block
constexpr size_t STRIP_PAIR_BYTES = 28 * 65536;        // the packed tiles above the diagonal blocks of an outer block
constexpr int STRIP_PACK_OUTER = 4;                    // outer blocks packed at a time (9 MB): one launch for every four strips
constexpr size_t STRIP_PACK_DIAG_BYTES = STRIP_PACK_OUTER * 8 * STRIP_DIAG_BYTES;
constexpr size_t STRIP_PACK_BYTES = STRIP_PACK_DIAG_BYTES + STRIP_PACK_OUTER * STRIP_PAIR_BYTES;
struct StripArgs {
    const float* S; int64_t lds_;   // working values [r x n]: weights (U form) or accumulators (R and hybrid forms); null: all zero
    const void* W; int64_t ldw; int wdtype; int w_vec;     // original weights (R and hybrid forms); w_vec: four at a time are aligned
    const float* diag; const float* pairs;                  // this outer block of the packed factor
    int64_t r, n, o0, o1;           // this outer block's columns
    int grid; int maxq;
    float* scales; int32_t* zeros; int64_t ngroups, group;
    int in_group;                   // group size if groups lie inside a block, else 0
    int64_t wide_group;             // group size if groups span 2, 4 or 8 blocks of an outer block, else 0
    uint8_t* codes; int64_t ldc;
    float* E; int64_t lde;          // out: -e (U form) or d = w - q of this outer block [r x 1024]; null: not wanted
    unsigned char* E_planes;        // ... as the pieces of the split products instead (split_planes.h); null: not wanted
    double* half_e2;
};
// Packs the outer blocks from column j_first on (a multiple of STRIP_PACK_OUTER * 1024) into STRIP_PACK_BYTES bytes: diagonal
// blocks first, the tiles of the outer blocks STRIP_PACK_DIAG_BYTES later.  M: what the later blocks of an outer block are
// updated with; D: the triangular blocks that are walked -- M's own (diag_dense = false) or dense 128 x 128 ones.
// with_pairs = false: outer blocks of one block.
int launch_pack_factor(const float* M, int64_t ldm, const float* D, int64_t ldd, bool diag_dense, int64_t n, int64_t j_first, bool with_pairs,
                       float* packed, hipStream_t s);
int launch_alg1_strip(bool rf, bool hybrid, const StripArgs& g, hipStream_t s);
// Ub[b] = R_bb^-1 for every 128 x 128 diagonal block of R (dense, identity outside a short last block).
int launch_invert_diag_blocks(const float* R, int64_t ldr, int64_t n, float* Ub, hipStream_t s);
// Rt[0:j0, block] = R[0:j0, block] U_bb for every column block (the part above the diagonal blocks; the rest of Rt is
// not written).
int launch_scale_column_blocks(const float* R, int64_t ldr, int64_t n, const float* Ub, float* Rt, int64_t ldt, hipStream_t s);

}  // namespace gptq
