// Step 3: Algorithm 1 -- column-by-column quantization in lazy blocks of B = 128 with error
// propagation (Section 3, Steps 1-3; Alg. 1), grids of Section 4 (Setup; grouping; "Extreme
// Quantization").
//
//   alg1_strip_kernel (quantize_strip.hip): the blocks of 128 columns of one outer block of 1024, in one launch -- the
//       column walk of every block and the rank-128 updates between them, a strip of rows per workgroup.  Outputs:
//       codes, the outer block's errors (r x 1024), per-row sum of e^2.
//   trailing update: W[:, later] -= E * U[block, later] for the columns beyond the outer block (rank 1024), the float32
//       matrix-core GEMM or the split products.
#include "quantize_common.h"

namespace gptq {

// One workgroup per row: convert the row and reduce min / max / max|.|.
template <typename T>
__global__ __launch_bounds__(256) void prepare_rows_kernel(const T* W, int64_t ldw, int64_t n, float* Wk, int64_t ldk,
                                                           int want_grid, int grid, float maxq, float* scales, int32_t* zeros) {
    const int64_t row = blockIdx.x;
    float lo = INFINITY, hi = -INFINITY, am = 0.f;
    for (int64_t k = threadIdx.x; k < n; k += 256) {
        const float v = to_f32<T>(W[row * ldw + k]);
        Wk[row * ldk + k] = v;
        lo = fminf(lo, v); hi = fmaxf(hi, v); am = fmaxf(am, fabsf(v));
    }
    if (!want_grid) return;
    __shared__ float slo[256], shi[256], sam[256];
    slo[threadIdx.x] = lo; shi[threadIdx.x] = hi; sam[threadIdx.x] = am;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            slo[threadIdx.x] = fminf(slo[threadIdx.x], slo[threadIdx.x + w]);
            shi[threadIdx.x] = fmaxf(shi[threadIdx.x], shi[threadIdx.x + w]);
            sam[threadIdx.x] = fmaxf(sam[threadIdx.x], sam[threadIdx.x + w]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        float sc; int zr;
        grid_from_range(grid, maxq, slo[0], shi[0], sam[0], sc, zr);
        scales[row] = sc; zeros[row] = zr;
    }
}

// Grid of one group that spans several blocks (group % 128 == 0): one wavefront per row over the
// current working weights W[:, j : j+g].
__global__ __launch_bounds__(64) void group_grid_kernel(const float* Wk, int64_t ldk, int64_t j, int64_t g, int grid, float maxq,
                                                        float* scales, int32_t* zeros, int64_t ngroups, int64_t gidx) {
    const int64_t row = blockIdx.x;
    float lo = INFINITY, hi = -INFINITY, am = 0.f;
    for (int64_t k = threadIdx.x; k < g; k += 64) {
        const float v = Wk[row * ldk + j + k];
        lo = fminf(lo, v); hi = fmaxf(hi, v); am = fmaxf(am, fabsf(v));
    }
    for (int off = 32; off > 0; off >>= 1) {
        lo = fminf(lo, __shfl_xor(lo, off));
        hi = fmaxf(hi, __shfl_xor(hi, off));
        am = fmaxf(am, __shfl_xor(am, off));
    }
    if (threadIdx.x == 0) {
        float sc; int zr;
        grid_from_range(grid, maxq, lo, hi, am, sc, zr);
        scales[row * ngroups + gidx] = sc; zeros[row * ngroups + gidx] = zr;
    }
}

// One workgroup per row: the per-row grid from the original weights, and the row of accumulators cleared.
template <typename T>
__global__ __launch_bounds__(256) void prepare_rows_rf_kernel(const T* W, int64_t ldw, int64_t n, float* S, int64_t lds_,
                                                              int want_grid, int grid, float maxq, float* scales, int32_t* zeros) {
    const int64_t row = blockIdx.x;
    float lo = INFINITY, hi = -INFINITY, am = 0.f;
    if (!want_grid) {                                       // grouped grids are taken block by block, from the current weights
        for (int64_t k = threadIdx.x; k < n; k += 256) S[row * lds_ + k] = 0.f;
        return;
    }
    for (int64_t k = threadIdx.x; k < n; k += 256) {
        const float v = to_f32<T>(W[row * ldw + k]);
        S[row * lds_ + k] = 0.f;
        lo = fminf(lo, v); hi = fmaxf(hi, v); am = fmaxf(am, fabsf(v));
    }
    __shared__ float slo[256], shi[256], sam[256];
    slo[threadIdx.x] = lo; shi[threadIdx.x] = hi; sam[threadIdx.x] = am;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            slo[threadIdx.x] = fminf(slo[threadIdx.x], slo[threadIdx.x + w]);
            shi[threadIdx.x] = fmaxf(shi[threadIdx.x], shi[threadIdx.x + w]);
            sam[threadIdx.x] = fmaxf(sam[threadIdx.x], sam[threadIdx.x + w]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        float sc; int zr;
        grid_from_range(grid, maxq, slo[0], shi[0], sam[0], sc, zr);
        scales[row] = sc; zeros[row] = zr;
    }
}

// Wq = scale * (code - zero)
__global__ __launch_bounds__(256) void dequant_kernel(const uint8_t* codes, int64_t ldc, const float* scales, const int32_t* zeros,
                                                      int64_t ngroups, int64_t gsize, int64_t n, float* Wq, int64_t ldq) {
    const int64_t row = blockIdx.x;
    for (int64_t k = threadIdx.x; k < n; k += 256) {
        const int64_t gi = k / gsize;
        const float sc = scales[row * ngroups + gi];
        const float zf = (float)zeros[row * ngroups + gi];
        Wq[row * ldq + k] = sc * ((float)codes[row * ldc + k] - zf);
    }
}

static bool group_supported(int64_t group) {
    if (group == 0) return true;
    if (group < 0) return false;
    if (group % QB == 0) return true;
    return group == 8 || group == 16 || group == 32 || group == 64;
}

// The factor form takes one grid per row, or groups that lie inside a block and are wide enough for the walk to be
// worth instantiating (32, 64, 128).
static bool factor_form_group_supported(int64_t group) { return group == 0 || group == 32 || group == 64 || group == 128; }

// Trailing updates beyond an outer block are deferred and applied as one rank-1024 GEMM.
static_assert(QOB == SPLIT_K, "the split products take exactly one outer block as K");

// The deferred rank-1024 updates go through the split-operand kernel (bf16 matrix cores, gemm_split.hip) when columns come in whole panels
// of 256.  `r` are the padded rows, so any row count above 128 qualifies.  They are the faster at every size (4096 x 1024 57 us
// against 70, 256 x 256 42 against 66) and the closer: relative error against 64-bit products 1.3e-7, 5.7e-7 in float32.
static bool split_shapes_ok(int64_t r, int64_t n) { return r >= 256 && r % 256 == 0 && n % 256 == 0 && n >= 2 * QOB; }

// Rows of the working matrix and of the error panels in the workspace: whole tiles of the deferred updates, so that a layer
// of any row count takes the large-tile kernels (3000 rows x 5120 columns: 190-250 us an update through the guarded
// kernel, 75-210 so).  Up to 128 rows one row of 128 x 128 tiles is enough, and half the memory.  The rows past r are never
// written by anything but these updates and never read by anything else.
static int64_t padded_rows(int64_t r) { return r >= 64 ? (int64_t)round_up((size_t)r, r <= 128 ? 128 : 256) : std::max<int64_t>(r, 1); }

struct QuantWs { size_t wk, e, pk, ub, rt, pa, pr, total; int64_t ldk, rows; bool split; };
static QuantWs quant_ws_layout(int64_t r, int64_t n, int64_t group) {
    QuantWs l;
    l.ldk = (int64_t)round_up((size_t)std::max<int64_t>(n, 1), 4);
    l.rows = padded_rows(r);
    l.wk = 0;
    size_t off = round_up((size_t)l.rows * l.ldk * sizeof(float), 256);
    l.e = off; off += 2 * round_up((size_t)l.rows * QOB * sizeof(float), 256);   // two error panels (look-ahead)
    l.pk = off; off += round_up(STRIP_PACK_BYTES, 256);                                             // four outer blocks of the factor as the strip kernel reads them
    const bool inner_groups = group != 0 && factor_form_group_supported(group);
    l.ub = off;                                                                                       // factor form with groups: every U_bb
    if (inner_groups) off += round_up((size_t)ceil_div(std::max<int64_t>(n, 1), QB) * QB * QB * sizeof(float), 256);
    l.rt = off;                                                                                       // ... and R with its column blocks scaled by them
    if (inner_groups) off += round_up((size_t)std::max<int64_t>(n, 1) * l.ldk * sizeof(float), 256);
    // split products (gemm_split.hip): the bf16 pieces of an error panel (every other one's lie in place of the two float32 panels) and of
    // an outer block's rows of U
    l.split = split_shapes_ok(l.rows, n);
    l.pa = l.pr = off;
    if (l.split) {
        l.pa = off; off += round_up(split_planes_bytes(l.rows), 256);
        l.pr = off; off += round_up(split_planes_bytes(n), 256);
    }
    l.total = off + 256;
    return l;
}

}  // namespace gptq

using namespace gptq;

extern "C" int gptq_trailing_update(float* W, int64_t ldw, const float* E, int64_t lde, const float* U, int64_t ldu,
                                    int64_t r, int64_t ncols, int64_t k, void* stream) {
    if (r < 0 || ncols < 0 || k < 0) return fail(GPTQ_ERR_INVALID_ARG, "trailing_update: negative size");
    if (r == 0 || ncols == 0 || k == 0) return GPTQ_OK;
    if (!W || !E || !U) return fail(GPTQ_ERR_INVALID_ARG, "trailing_update: null pointer");
    if (ldw < ncols || lde < k || ldu < ncols) return fail(GPTQ_ERR_INVALID_ARG, "trailing_update: leading dimension smaller than the row length");
    if (!aligned(W, 16) || !aligned(E, 16) || !aligned(U, 16) || ldw % 4 || lde % 4 || ldu % 4)
        return fail(GPTQ_ERR_INVALID_ARG, "trailing_update: W, E and U must be 16-byte aligned with leading dimensions that are multiples of 4");
    GemmF32 g{};
    g.A = E; g.lda = lde; g.B = U; g.ldb = ldu; g.C = W; g.ldc = ldw;
    g.M = r; g.N = ncols; g.K = k; g.alpha = -1.f; g.b_is_nk = false; g.overwrite = false;
    return launch_gemm_f32(g, static_cast<hipStream_t>(stream));
}

extern "C" size_t gptq_quantize_layer_workspace_bytes(int64_t r, int64_t n, int block, int64_t group) {
    (void)block;
    if (r < 0 || n < 0) return 0;
    return quant_ws_layout(r, n, group).total;
}

// Both forms of Alg. 1 share validation, blocking and look-ahead.  rf = false: `U` is Cholesky((H + lambda I)^-1)^T,
// the working weights are updated (W -= E U).  rf = true: `U` is R with H + lambda I = R R^T, the accumulators are
// updated (S += D R) and the weights are read from the caller's W as they are (one grid per row only).
static int alg1_run(bool rf, const void* W, int wdtype, int64_t ldw, int64_t r, int64_t n,
                    const float* U, int64_t ldu,
                    int bits, int grid, int block, int64_t group,
                    uint8_t* codes, int64_t ldc, float* scales, int32_t* zeros,
                    float* Wq, int64_t ldq, double* half_E2_rows,
                    void* ws, size_t ws_bytes, void* stream) {
    if (r < 0 || n < 0) return fail(GPTQ_ERR_INVALID_ARG, "quantize_layer: negative size");
    if (grid != GPTQ_GRID_MINMAX && grid != GPTQ_GRID_TERNARY) return fail(GPTQ_ERR_INVALID_ARG, "quantize_layer: unknown grid %d", grid);
    if (grid == GPTQ_GRID_MINMAX && (bits < 2 || bits > 4)) return fail(GPTQ_ERR_INVALID_ARG, "quantize_layer: bits must be 2, 3 or 4 (got %d)", bits);
    if (wdtype != GPTQ_F16 && wdtype != GPTQ_BF16 && wdtype != GPTQ_F32) return fail(GPTQ_ERR_INVALID_ARG, "quantize_layer: unknown wdtype %d", wdtype);
    if (block <= 0) return fail(GPTQ_ERR_INVALID_ARG, "quantize_layer: block must be positive");
    if (block != QB) return fail(GPTQ_ERR_UNSUPPORTED, "quantize_layer: only block = 128 is built (got %d)", block);
    if (group < 0) return fail(GPTQ_ERR_INVALID_ARG, "quantize_layer: negative group");
    if (group > 0 && n % group) return fail(GPTQ_ERR_INVALID_ARG, "quantize_layer: n must be a multiple of the group size");
    if (group > 0 && (QB % group) && (group % QB)) return fail(GPTQ_ERR_INVALID_ARG, "quantize_layer: a group must not straddle a block end (need 128 %% g == 0 or g %% 128 == 0)");
    if (!group_supported(group)) return fail(GPTQ_ERR_UNSUPPORTED, "quantize_layer: group size %lld not built (8, 16, 32, 64 or a multiple of 128)", (long long)group);
    if (rf && !factor_form_group_supported(group))
        return fail(GPTQ_ERR_UNSUPPORTED, "quantize_layer_from_factor: one grid per row or groups of 32, 64 or 128 columns (got %lld); a group's grid "
                                          "is taken from the current weights, which this form rebuilds one block at a time: use "
                                          "gptq_damp_cholesky_inverse + gptq_quantize_layer", (long long)group);
    if (r == 0 || n == 0) return GPTQ_OK;
    if (!W || !U || !codes || !scales || !zeros) return fail(GPTQ_ERR_INVALID_ARG, "quantize_layer: null pointer");
    if (ldw < n || ldu < n || ldc < n || (Wq && ldq < n)) return fail(GPTQ_ERR_INVALID_ARG, "quantize_layer: leading dimension smaller than n");
    if (!aligned(U, 16) || ldu % 4) return fail(GPTQ_ERR_INVALID_ARG, "quantize_layer: U must be 16-byte aligned with ldu %% 4 == 0");
    const QuantWs lay = quant_ws_layout(r, n, group);
    if (!ws || !aligned(ws, 256) || ws_bytes < lay.total) return fail(GPTQ_ERR_WORKSPACE, "quantize_layer: workspace missing, misaligned or too small");
    if (r > 0x7fffffffLL) return fail(GPTQ_ERR_UNSUPPORTED, "quantize_layer: too many rows");

    hipStream_t s = static_cast<hipStream_t>(stream);
    char* base = static_cast<char*>(ws);
    float* Wk = reinterpret_cast<float*>(base + lay.wk);
    float* Ebuf[2] = {reinterpret_cast<float*>(base + lay.e),
                      reinterpret_cast<float*>(base + lay.e + round_up((size_t)lay.rows * QOB * sizeof(float), 256))};
    const int64_t rows = lay.rows;
    const int maxq = (grid == GPTQ_GRID_TERNARY) ? 2 : ((1 << bits) - 1);
    const int64_t ngroups = group ? n / group : 1;
    const int want_grid = group == 0;

    if (rf) {
        switch (wdtype) {
            case GPTQ_F16:
                hipLaunchKernelGGL(prepare_rows_rf_kernel<_Float16>, dim3((unsigned)r), dim3(256), 0, s, static_cast<const _Float16*>(W), ldw, n, Wk, lay.ldk, want_grid, grid, (float)maxq, scales, zeros);
                break;
            case GPTQ_BF16:
                hipLaunchKernelGGL(prepare_rows_rf_kernel<__bf16>, dim3((unsigned)r), dim3(256), 0, s, static_cast<const __bf16*>(W), ldw, n, Wk, lay.ldk, want_grid, grid, (float)maxq, scales, zeros);
                break;
            default:
                hipLaunchKernelGGL(prepare_rows_rf_kernel<float>, dim3((unsigned)r), dim3(256), 0, s, static_cast<const float*>(W), ldw, n, Wk, lay.ldk, want_grid, grid, (float)maxq, scales, zeros);
        }
    } else
    switch (wdtype) {
        case GPTQ_F16:
            hipLaunchKernelGGL(prepare_rows_kernel<_Float16>, dim3((unsigned)r), dim3(256), 0, s, static_cast<const _Float16*>(W), ldw, n, Wk, lay.ldk, want_grid, grid, (float)maxq, scales, zeros);
            break;
        case GPTQ_BF16:
            hipLaunchKernelGGL(prepare_rows_kernel<__bf16>, dim3((unsigned)r), dim3(256), 0, s, static_cast<const __bf16*>(W), ldw, n, Wk, lay.ldk, want_grid, grid, (float)maxq, scales, zeros);
            break;
        default:
            hipLaunchKernelGGL(prepare_rows_kernel<float>, dim3((unsigned)r), dim3(256), 0, s, static_cast<const float*>(W), ldw, n, Wk, lay.ldk, want_grid, grid, (float)maxq, scales, zeros);
    }
    GPTQ_LAUNCH_CHECK();
    const bool hybrid = rf && group != 0;
    float* Ub = reinterpret_cast<float*>(base + lay.ub);
    // The matrix the deferred updates multiply with: U, R, or -- factor form with groups -- Rt = R with every column block
    // scaled by the inverse of its diagonal block (made here, once), so that the accumulators of a block hold s R_bb^-1.
    const float* Bm = U;
    int64_t ldb = ldu;
    if (hybrid) {
        float* Rt = reinterpret_cast<float*>(base + lay.rt);
        if (int rc = launch_invert_diag_blocks(U, ldu, n, Ub, s)) return rc;
        if (int rc = launch_scale_column_blocks(U, ldu, n, Ub, Rt, lay.ldk, s)) return rc;
        Bm = Rt; ldb = lay.ldk;
    }

    // Lazy batching at two levels (Section 3, Step 2 applied twice): inside an outer block of 1024 columns
    // each 128-column block updates only the rest of the outer block (rank 128, inside the strip kernel); the columns
    // beyond it get one rank-1024 update per outer block.  Same sums as Alg. 1, associated differently.
    const int64_t ob = alg1_outer_block(group);
    // With the split products the strip kernel writes the error panel as their pieces, in turn into two places (the room of the float32
    // panels is one of them), and the pieces of an outer block's rows of U are made ahead on the helper stream.  One decision for the call.
    const bool split = lay.split && ob == QOB && n > QOB && split_pays((rows / 256) * (QOB / 256), true);
    unsigned char* Pe[2] = {reinterpret_cast<unsigned char*>(base + lay.pa), reinterpret_cast<unsigned char*>(base + lay.e)};
    unsigned char* Pu = reinterpret_cast<unsigned char*>(base + lay.pr);
    // Look-ahead: after an outer block is quantized, the columns of the next outer block are updated first, on
    // the caller's stream, which goes straight on to quantize them (short, serial kernels); all columns
    // beyond are updated on the helper stream meanwhile.  The two updates and the next block's kernels touch
    // disjoint columns of the weights; the error panel E alternates between two buffers because the helper's
    // GEMM still reads one while the next block fills the other.
    HelperStreams ts;
    if (int rc = ts.open(s, n > 2 * ob ? 1 : 0)) return rc;        // up to two outer blocks nothing is updated beyond the next one
    hipStream_t s2 = ts.side[0];
    hipEvent_t rest_done = nullptr;         // the helper stream's last trailing update, if one is pending
    hipEvent_t factor_split = nullptr;      // ... and the pieces of U's rows for the updates that come next
    if (split) {
        if (int rc = launch_split_cols(Bm + ob, ldb, n - ob, Pu, s2)) return rc;
        if (int rc = ts.mark(s2, &factor_split)) return rc;
    }
    const bool outer_groups = group > QB && (ob == QB || group > QOB);      // groups that the strip kernel does not see whole
    float* packed = reinterpret_cast<float*>(base + lay.pk);
    StripArgs strip{};
    strip.lds_ = lay.ldk;
    strip.W = W; strip.ldw = ldw; strip.wdtype = wdtype;
    strip.w_vec = ldw % 4 == 0 && aligned(W, wdtype == GPTQ_F32 ? 16 : 8);
    strip.r = r; strip.n = n; strip.grid = grid; strip.maxq = maxq;
    strip.scales = scales; strip.zeros = zeros; strip.ngroups = ngroups; strip.group = group;
    strip.in_group = group <= QB ? (int)group : 0;
    strip.wide_group = (group > QB && !outer_groups) ? group : 0;
    strip.codes = codes; strip.ldc = ldc; strip.lde = QOB; strip.half_e2 = half_E2_rows;
    int eb = 0;
    for (int64_t o0 = 0; o0 < n; o0 += ob, eb ^= 1) {
        const int64_t o1 = std::min<int64_t>(o0 + ob, n);
        float* E = Ebuf[eb];
        // The grid of a group wider than an outer block is taken from all of its columns as they stand now.  Those beyond
        // this outer block are kept current by the helper stream: its last update has to be in.
        if (outer_groups && o0 % group == 0) {
            if (o0 + group > o1) { if (int rc = ts.wait(s, rest_done)) return rc; }
            hipLaunchKernelGGL(group_grid_kernel, dim3((unsigned)r), dim3(64), 0, s, (const float*)Wk, lay.ldk, o0, group, grid, (float)maxq, scales, zeros, ngroups, o0 / group);
            GPTQ_LAUNCH_CHECK();
        }
        const int64_t in_pack = o0 % (STRIP_PACK_OUTER * QOB);
        if (in_pack == 0)
            if (int rc = launch_pack_factor(Bm, ldb, hybrid ? Ub : U, ldu, hybrid, n, o0, ob == QOB, packed, s)) return rc;
        strip.diag = packed + (in_pack / QB) * (int64_t)(STRIP_DIAG_BYTES / sizeof(float));
        strip.pairs = packed + STRIP_PACK_DIAG_BYTES / sizeof(float) + (in_pack / QOB) * (int64_t)(STRIP_PAIR_BYTES / sizeof(float));
        strip.o0 = o0; strip.o1 = o1;
        strip.S = (rf && o0 == 0) ? nullptr : Wk;               // the accumulators start at zero
        strip.E = o1 < n && !split ? E : nullptr;
        strip.E_planes = o1 < n && split ? Pe[eb] : nullptr;
        if (int rc = launch_alg1_strip(rf, hybrid, strip, s)) return rc;
        if (o1 < n) {
            const int64_t o2 = std::min<int64_t>(o1 + ob, n);
            hipEvent_t quantized = nullptr;
            if (int rc = ts.mark(s, &quantized)) return rc;
            if (int rc = ts.wait(s, rest_done)) return rc;      // it wrote the columns from o1 on
            rest_done = nullptr;
            const float alpha = 1.f;                 // the U form's panel holds -e
            SplitGemm sg{};
            sg.A_planes = Pe[eb]; sg.B_planes = Pu;
            sg.ldc = lay.ldk; sg.alpha = alpha; sg.M = rows; sg.K = SPLIT_K;
            GemmF32 g{};
            g.A = E; g.lda = QOB; g.B = Bm + o0 * ldb + o1; g.ldb = ldb; g.C = Wk + o1; g.ldc = lay.ldk;
            g.M = rows; g.N = o2 - o1; g.K = o1 - o0; g.alpha = alpha; g.b_is_nk = false; g.overwrite = false;
            hipEvent_t next_done = nullptr;
            if (split) {
                if (int rc = ts.wait(s, factor_split)) return rc;
                sg.C = Wk + o1; sg.N = o2 - o1;
                if (int rc = launch_gemm_split(sg, s)) return rc;
                if (int rc = ts.mark(s, &next_done)) return rc;
            } else {
                if (int rc = launch_gemm_f32(g, s)) return rc;
            }
            if (o2 < n) {
                if (int rc = ts.wait(s2, quantized)) return rc;
                if (split) {
                    sg.b_panel0 = (int)((o2 - o1) / 256);
                    sg.C = Wk + o2; sg.N = n - o2;
                    if (int rc = launch_gemm_split(sg, s2)) return rc;
                } else {
                    g.B = Bm + o0 * ldb + o2; g.C = Wk + o2; g.N = n - o2;
                    if (int rc = launch_gemm_f32(g, s2)) return rc;
                }
                if (int rc = ts.mark(s2, &rest_done)) return rc;
                if (split) {
                    // the next outer block's, into the same place: both of its readers are through
                    if (int rc = ts.wait(s2, next_done)) return rc;
                    if (int rc = launch_split_cols(Bm + o1 * ldb + o2, ldb, n - o2, Pu, s2)) return rc;
                    if (int rc = ts.mark(s2, &factor_split)) return rc;
                }
            }
        }
    }
    if (Wq) {
        hipLaunchKernelGGL(dequant_kernel, dim3((unsigned)r), dim3(256), 0, s, (const uint8_t*)codes, ldc, (const float*)scales, (const int32_t*)zeros,
                           ngroups, group ? group : n, n, Wq, ldq);
        GPTQ_LAUNCH_CHECK();
    }
    return GPTQ_OK;
}

extern "C" int gptq_quantize_layer(const void* W, int wdtype, int64_t ldw, int64_t r, int64_t n,
                                   const float* U, int64_t ldu,
                                   int bits, int grid, int block, int64_t group,
                                   uint8_t* codes, int64_t ldc, float* scales, int32_t* zeros,
                                   float* Wq, int64_t ldq, double* half_E2_rows,
                                   void* ws, size_t ws_bytes, void* stream) {
    return alg1_run(false, W, wdtype, ldw, r, n, U, ldu, bits, grid, block, group, codes, ldc, scales, zeros, Wq, ldq,
                    half_E2_rows, ws, ws_bytes, stream);
}

extern "C" int gptq_quantize_layer_from_factor_supports(int64_t group) { return factor_form_group_supported(group) ? 1 : 0; }

extern "C" int gptq_quantize_layer_from_factor(const void* W, int wdtype, int64_t ldw, int64_t r, int64_t n,
                                               const float* R, int64_t ldr,
                                               int bits, int grid, int block, int64_t group,
                                               uint8_t* codes, int64_t ldc, float* scales, int32_t* zeros,
                                               float* Wq, int64_t ldq, double* half_E2_rows,
                                               void* ws, size_t ws_bytes, void* stream) {
    return alg1_run(true, W, wdtype, ldw, r, n, R, ldr, bits, grid, block, group, codes, ldc, scales, zeros, Wq, ldq,
                    half_E2_rows, ws, ws_bytes, stream);
}
