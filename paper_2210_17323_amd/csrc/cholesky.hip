// Step 2: lambda = percdamp * mean(diag H); U = Cholesky((H + lambda I)^-1)^T
// (Section 3, Step 3 and Alg. 1, third statement).
//
// Route: factor H + lambda I = R R^T with R upper triangular -- a Cholesky factorisation that starts at
// the last column and moves backwards -- then invert the triangle, U = R^-1.  (H + lambda I)^-1 =
// R^-T R^-1 = U^T U and the Cholesky factor with positive diagonal is unique, so this U is the
// matrix Alg. 1 asks for, at half the flops of "Cholesky, invert, Cholesky again" and without ever
// forming the explicit inverse.
//
// Two-level blocking (inner blocks of 128 columns, outer blocks of 1024), result in place in the upper triangle.
//
// Factorisation, outer blocks o last .. first:
//     R_oo = reverse-Cholesky of the 1024 x 1024 diagonal block, inner blocks b last .. first, and every R_bb^-1  (one launch, chol_chain.hip)
//     R[0:o0, o] = H[0:o0, o] R_oo^-T              (strips of rows, one launch, chol_strip.hip)
//     H[0:o0, 0:o0] -= R[0:o0, o] R[0:o0, o]^T     (rank 1024, carries the flops)
// The chain of an outer block takes 184 us while nothing else runs, up to 310 beside the updates of a 12288 x 12288 matrix, whose workgroups
// hold the CUs it has to start on.  With two launches per block of 128 columns, 8 x (28 + 15) us alone and 8 x (36 + 26) beside the updates, and
// with the whole panel and the update of the next 1024 columns between two chains, n = 12288 took 9.26 ms and the inverse at
// n = 5000 3.41; 6.76 and 2.23 before the updates and the inverse's products went to the split products, 5.3 and 1.90 since.
//
//   one outer block behind, on a stream of its own (only when the inverse is wanted): U_oo = R_oo^-1, kept dense for the
//     inverse (chol_strip.hip).
//
// Triangular inverse (right-looking, outer block columns k first .. last), with the U_kk kept from the factorisation:
//     T = -U_kk R[k, right of k] ;  U[above k, right of k] += U[above k, k] T ;  row block k <- T
//     U[above k, k] <- U[above k, k] U_kk ;  diagonal block <- U_kk
// Every long product has K = 1024 and an output of (rows above) x (columns to the right): many tiles at every k.
#include "chol_chain.h"
#include "chol_strip.h"
#include "common.h"

#include <mutex>

namespace gptq {

constexpr int NB = 128;

// One workgroup: mean of the diagonal in float64, lambda in float32, add it to the diagonal.
__global__ __launch_bounds__(1024) void damp_kernel(float* H, int64_t ld, int64_t n, float percdamp, int* info, int* flags) {
    __shared__ double part[1024];
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 1024) s += (double)H[i * ld + i];
    part[threadIdx.x] = s;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    const float lambda = percdamp * (float)(part[0] / (double)n);
    for (int64_t i = threadIdx.x; i < n; i += 1024) H[i * ld + i] += lambda;
    if (threadIdx.x == 0) *info = 0;
    if (threadIdx.x < CHAIN_FLAG_BYTES / sizeof(int)) flags[threadIdx.x] = 0;
}

// dst[rows x cols] (ld_dst) = src[rows x cols] (ld_src), optionally only the upper triangle of a
// square block (strictly lower part written as zero).
__global__ __launch_bounds__(256) void copy_block_kernel(float* dst, int64_t ld_dst, const float* src, int64_t ld_src,
                                                         int64_t rows, int cols, int upper_square) {
    const int64_t total = rows * cols;
    for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < total; q += (int64_t)gridDim.x * 256) {
        const int64_t i = q / cols;
        const int k = (int)(q % cols);
        float v = src[i * ld_src + k];
        if (upper_square && k < i) v = 0.f;
        dst[i * ld_dst + k] = v;
    }
}

// dst[rows x cols] = src[rows x cols]; both 16-byte aligned with leading dimensions and cols that are multiples of 4
__global__ __launch_bounds__(256) void copy2d_kernel(float* dst, int64_t ld_dst, const float* src, int64_t ld_src, int64_t rows, int64_t cols4) {
    const int64_t total = rows * cols4;
    for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < total; q += (int64_t)gridDim.x * 256) {
        const int64_t i = q / cols4, c = q - i * cols4;
        reinterpret_cast<float4*>(dst + i * ld_dst)[c] = reinterpret_cast<const float4*>(src + i * ld_src)[c];
    }
}

__global__ __launch_bounds__(256) void fill_zero_kernel(float4* p, int64_t count4) {
    for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < count4; q += (int64_t)gridDim.x * 256)
        p[q] = make_float4(0.f, 0.f, 0.f, 0.f);
}

__global__ __launch_bounds__(256) void zero_lower_kernel(float* H, int64_t ld, int64_t n) {
    const int64_t row = blockIdx.x;
    for (int64_t k = threadIdx.x; k < row; k += 256) H[row * ld + k] = 0.f;
}

}  // namespace gptq

using namespace gptq;

namespace {
constexpr int OB = 1024;     // outer block: rank-1024 updates keep the big GEMMs compute-bound and their tiles long
static_assert(OB == SPLIT_K, "the split products take exactly one outer block as K");
// A rank-1024 update goes through the split-operand kernel (gemm_split.hip) above the sizes that the variant without a workspace takes, which
// has no planes and gives the same bits; with the last outer block's narrower panel too, whose K is no multiple of anything (in float32 that
// is the guarded kernel, 200 us an update and 189 for the last column block of the inverse at n = 5000).  At 4096 channels the split
// products would save 5 % of the factorisation and 10 % of the inverse.
constexpr int64_t SPLIT_ABOVE = GPTQ_NOALLOC_MAX_N;

struct CholWs { float* dinv; float* T; float* T2; int64_t ld2; float* Uoo; float* tri; float* tri2; unsigned char* planes; unsigned char* planes2; int* flags; size_t total; };
CholWs chol_ws_layout(void* ws, int64_t n, bool with_split = true) {
    const size_t n1 = (size_t)std::max<int64_t>(n, 1);
    const size_t nblk = (size_t)ceil_div((int64_t)n1, NB), nouter = (size_t)ceil_div((int64_t)n1, OB);
    size_t off = 0;
    CholWs l{};
    // with ws == nullptr only the total is wanted: no pointer is formed (arithmetic on a null pointer is undefined)
    uintptr_t base = reinterpret_cast<uintptr_t>(ws);
    auto at = [&](size_t bytes) { const size_t o = off; off += round_up(bytes, 256); return ws ? reinterpret_cast<void*>(base + o) : nullptr; };
    l.ld2 = (int64_t)round_up(n1, 4);
    l.dinv = static_cast<float*>(at(nblk * NB * NB * sizeof(float)));        // R_bb^-1, dense
    l.T = static_cast<float*>(at(n1 * OB * sizeof(float)));                  // a column panel [n x 1024]; the chain's scratch, 4 MiB (with T2 and Uoo, idle then, where n < 1024)
    l.T2 = static_cast<float*>(at((size_t)OB * l.ld2 * sizeof(float)));      // a row panel [1024 x n]
    l.Uoo = static_cast<float*>(at(nouter * OB * OB * sizeof(float)));       // U_oo of every outer block, dense
    l.tri = static_cast<float*>(at(TRIANGLE_WORDS * sizeof(float)));         // an outer block of R packed for its inverse
    l.tri2 = static_cast<float*>(at(TRIANGLE_WORDS * sizeof(float)));        // ... and for the rows above it (every other one)
    if (with_split && (int64_t)n1 >= 2 * OB) {                               // split products: bf16 pieces of a column panel
        l.planes = static_cast<unsigned char*>(at(split_planes_bytes((int64_t)n1)));
        l.planes2 = static_cast<unsigned char*>(at(split_planes_bytes((int64_t)n1)));      // ... and of a row block (the inverse)
    }
    l.flags = static_cast<int*>(at(CHAIN_FLAG_BYTES));                       // of the chain's workgroups
    l.total = off;
    return l;
}
}  // namespace

extern "C" size_t gptq_damp_cholesky_inverse_workspace_bytes(int64_t n) {
    return chol_ws_layout(nullptr, n < 0 ? 0 : n).total;
}

// Host-side checks shared by the entry points; 1 = nothing to do (n == 0).
static int chol_check_args(const float* H, int64_t ld, int64_t n, float percdamp, const int* info_dev, int* rc) {
    *rc = GPTQ_OK;
    if (n < 0) { *rc = fail(GPTQ_ERR_INVALID_ARG, "damp_cholesky_inverse: negative size"); return 1; }
    if (!info_dev) { *rc = fail(GPTQ_ERR_INVALID_ARG, "damp_cholesky_inverse: info_dev is null"); return 1; }
    if (n == 0) return 1;
    if (!H) { *rc = fail(GPTQ_ERR_INVALID_ARG, "damp_cholesky_inverse: H is null"); return 1; }
    if (ld < n || ld % 4 || !aligned(H, 16)) {
        *rc = fail(GPTQ_ERR_INVALID_ARG, "damp_cholesky_inverse: need ld >= n, ld %% 4 == 0 and a 16-byte aligned H");
        return 1;
    }
    if (!(percdamp >= 0.f)) { *rc = fail(GPTQ_ERR_INVALID_ARG, "damp_cholesky_inverse: percdamp must be >= 0"); return 1; }
    return 0;
}

// The whole of step 2 on validated arguments.  `ws` holds chol_ws_layout(n).total bytes; nothing in it has to be
// initialised (every region is written in this call before it is read).  lookahead = false keeps all work on `s`
// (the host code below enqueues in an order that respects every dependence, so one stream is always valid).
// want_inverse = false stops after the factorisation: H holds R (upper triangular, zeros below) with H + lambda I = R R^T.
static int chol_run(float* H, int64_t ld, int64_t n, float percdamp, void* ws, int* info_dev, hipStream_t s, bool lookahead,
                    bool want_inverse = true, bool with_split = true) {
    const CholWs w = chol_ws_layout(ws, n, with_split);
    float* dinv = w.dinv;
    hipLaunchKernelGGL(damp_kernel, dim3(1), dim3(1024), 0, s, H, ld, n, percdamp, info_dev, w.flags);
    GPTQ_LAUNCH_CHECK();

    // C (+)= alpha A op(B) on stream st
    struct Opt { bool nk = false, overwrite = false, upper = false, atri = false, btri = false; };
    auto gemm_on = [&](hipStream_t st, const float* A, int64_t lda, const float* B, int64_t ldb, float* C, int64_t ldc,
                       int64_t M, int64_t N, int64_t K, float alpha, const Opt& o) -> int {
        GemmF32 g{};
        g.A = A; g.lda = lda; g.B = B; g.ldb = ldb; g.C = C; g.ldc = ldc; g.M = M; g.N = N; g.K = K; g.alpha = alpha;
        g.b_is_nk = o.nk; g.overwrite = o.overwrite; g.upper_only = o.upper;
        g.a_upper_tri = o.atri; g.b_upper_tri = o.btri;
        return launch_gemm_f32(g, st);
    };
    auto copy2d = [&](hipStream_t st, float* dst, int64_t ld_dst, const float* src, int64_t ld_src, int64_t rows, int64_t cols) -> int {
        if (rows <= 0 || cols <= 0) return GPTQ_OK;
        if (cols % 4 == 0 && ld_dst % 4 == 0 && ld_src % 4 == 0 && aligned(dst, 16) && aligned(src, 16)) {
            const int64_t total4 = rows * (cols / 4);
            hipLaunchKernelGGL(copy2d_kernel, dim3((unsigned)std::min<int64_t>(ceil_div(total4, 256), 2048)), dim3(256), 0, st, dst, ld_dst, src, ld_src, rows, cols / 4);
        } else {
            hipLaunchKernelGGL(copy_block_kernel, dim3((unsigned)std::min<int64_t>(ceil_div(rows * cols, 256), 2048)), dim3(256), 0, st, dst, ld_dst, src, ld_src, rows, (int)cols, 0);
        }
        GPTQ_LAUNCH_CHECK();
        return GPTQ_OK;
    };
    const int64_t nouter = ceil_div(n, OB);
    // The products of the inverse as split products: the column blocks' pieces lie in turn in the planes of the factorisation and in the
    // two float32 panels, which have room for those of a diagonal block's inverse behind them (from 4096 channels on always).  The pieces of a
    // column block are made once, for the update and for the product with U_kk, which with overwriting needs no copy back: that product was 70
    // to 150 us of float32 on the other stream, which ended last, and T of the first outer block 50 us before the inverse could start.
    // Inverse, us, with the update alone split / all: n = 5000 2090 / 1900, 6144 2770 / 2510, 8192 4260 / 4090, 12288 9920 / 9500; error
    // against 64 bits at n = 5000 4.1e-7 / 3.2e-7.
    unsigned char* const panels = reinterpret_cast<unsigned char*>(w.T);
    const size_t panel_planes = round_up(split_planes_bytes((nouter - 1) * OB), 256);
    const bool inverse_split = want_inverse && w.planes && nouter > 1 && split_pays(4 * (nouter - 1), n > SPLIT_ABOVE) &&
                               panel_planes + split_planes_bytes(OB) <= (size_t)(reinterpret_cast<unsigned char*>(w.Uoo) - panels);
    unsigned char* const column_planes[2] = {w.planes, panels};
    unsigned char* const diag_planes = panels + panel_planes;
    HelperStreams ts;
    if (int rc = ts.open(s, lookahead && nouter > 1 ? (want_inverse ? 3 : 2) : 0)) return rc;
    hipStream_t s2 = ts.side[0];    // rank-1024 updates left of the next outer block but one
    hipStream_t s4 = ts.side[1];    // the rows above, and the update of the columns of the next outer block but one
    hipStream_t s3 = ts.side[2];    // one outer block behind the factorisation's chain: U_oo and its product

    // ---- H + lambda I = R R^T, from the last column backwards.  Two levels: inside an outer block of 1024 columns the
    //      rank-128 updates touch only that block's columns; the rest of the matrix gets one rank-1024 update per block.
    //
    //      Look-ahead: the next chain waits for one thing only, the update of its own 1024 x 1024 block, which needs 1024 rows of this
    //      outer block's panel.  Those rows and that update follow the chain on the caller's stream; the rows above and every other update
    //      run beside the next chain, the columns that are wanted next and the rest on streams of their own, so that
    //      the rows above the next outer block do not wait for the rest either.  (What main waits for was behind everything of the outer
    //      block but one before on s4, so the packed block it is about to overwrite has been read.)
    hipEvent_t strip_done = nullptr;    // s4: the last update of the columns of the next outer block but one, rows above it
    hipEvent_t rest_done = nullptr;     // s2: the last update of everything left of those
    for (int64_t o = nouter - 1; o >= 0; --o) {
        const int64_t o0 = o * OB, o1 = std::min<int64_t>(o0 + OB, n), ow = o1 - o0;
        const int64_t p0 = o0 - OB;                      // outer blocks start at multiples of OB
        // the packed outer block, in turn in two places: the one before may still be read.  The second place is behind the chain's
        // scratch in the column panel, which has more than 2 OB rows where a second one is wanted.
        float* packed_block = o == 0 ? nullptr : ((o & 1) || nouter <= 2 ? w.tri2 : w.T + (int64_t)OB * OB);
        float* Ublk = w.Uoo + o * (int64_t)OB * OB;      // U_oo = R_oo^-1 [ow x ow], leading dimension OB, for the inverse
        if (int rc = launch_chol_chain(H, ld, o0, (int)ow, dinv + o * (int64_t)(OB / NB) * NB * NB, w.T, packed_block, w.flags, (int)(nouter - o), info_dev, s)) return rc;
        if (want_inverse) {
            // One outer block behind, on its own stream: U_oo = R_oo^-1, dense with zeros below the diagonal (the products that
            // read it rely on them), and R[o, right] <- -U_oo R[o, right], which is what the inverse below needs of this row
            // block.  Both are final here, the last to read them are the updates behind the outer block before, and the
            // product depends on nothing the inverse computes, so it is taken off the inverse's serial path.
            hipEvent_t chain = nullptr;
            if (int rc = ts.mark(s, &chain)) return rc;
            hipLaunchKernelGGL(fill_zero_kernel, dim3(256), dim3(256), 0, s3, reinterpret_cast<float4*>(Ublk), (int64_t)OB * OB / 4);
            GPTQ_LAUNCH_CHECK();
            if (int rc = ts.wait(s3, chain)) return rc;
            if (int rc = launch_pack_triangle(H, ld, n, dinv, o, w.tri, s3)) return rc;
            if (int rc = launch_triangle_inverse(w.tri, n, o, Ublk, s3)) return rc;
            if (o1 < n && o == 0 && inverse_split) {
                // the last one, which the inverse waits for; the planes' readers are behind the chain just walked
                if (int rc = launch_split_rows(Ublk, OB, ow, w.planes, s3)) return rc;
                if (int rc = launch_split_cols(H + o1, ld, n - o1, w.planes2, s3)) return rc;
                SplitGemm sg{};
                sg.A_planes = w.planes; sg.B_planes = w.planes2;
                sg.C = H + o1; sg.ldc = ld; sg.alpha = -1.f; sg.M = ow; sg.N = n - o1; sg.K = OB; sg.overwrite = true;
                if (int rc = launch_gemm_split(sg, s3)) return rc;
            } else if (o1 < n) {
                Opt a; a.overwrite = true; a.atri = true;
                if (int rc = gemm_on(s3, Ublk, OB, H + o0 * ld + o1, ld, w.T2, w.ld2, ow, n - o1, ow, -1.f, a)) return rc;
                if (int rc = ts.wait(s3, strip_done)) return rc;
                if (int rc = ts.wait(s3, rest_done)) return rc;
                if (int rc = copy2d(s3, H + o0 * ld + o1, ld, w.T2, w.ld2, ow, n - o1)) return rc;
            }
        }
        if (o0 == 0) break;
        // R[p0:o0, o] = H[p0:o0, o] R_oo^-T, a strip of rows per workgroup (chol_strip.hip), then H[p0:o0, p0:o0]
        hipEvent_t chained = nullptr;
        if (int rc = ts.mark(s, &chained)) return rc;
        if (int rc = ts.wait(s, strip_done)) return rc;
        if (int rc = launch_triangle_panel(H + p0 * ld + o0, ld, OB, packed_block, n, o, s)) return rc;
        hipEvent_t rows_done = nullptr;
        if (int rc = ts.mark(s, &rows_done)) return rc;
        if (p0 > 0) {
            if (int rc = ts.wait(s4, chained)) return rc;
            if (int rc = launch_triangle_panel(H + o0, ld, p0, packed_block, n, o, s4)) return rc;
        }
        const hipEvent_t before = rest_done;
        if (int rc = ts.wait(s, before)) return rc;
        if (int rc = launch_next_block_update(H + p0 * ld + p0, ld, H + p0 * ld + o0, ld, ow, s)) return rc;
        if (p0 == 0) continue;
        // H[0:p0, 0:o0] -= R[0:p0, o] R[0:o0, o]^T (rank 1024, upper tiles), the columns [p0, o0) on one stream and the square left of
        // them on the other.  Large updates multiply the bf16 pieces of the panel R[0:o0, o] (gemm_split.hip): one split of it serves both
        // parts, as row operand and as column operand; the pieces of two panels take turns, since the square of the outer block before
        // may still be read.
        if (int rc = ts.wait(s4, rows_done)) return rc;
        // (the two run beside each other: what counts is whether they fill the chip together)
        const bool split = w.planes && split_pays((p0 / 256) * (OB / 256) + (p0 / 256) * (p0 / 256 + 1) / 2, n > SPLIT_ABOVE);
        unsigned char* planes = (o & 1) ? w.planes2 : w.planes;
        if (split)
            if (int rc = launch_split_rows(H + o0, ld, o0, planes, s4, ow)) return rc;
        hipEvent_t panel = nullptr;
        if (int rc = ts.mark(s4, &panel)) return rc;
        if (int rc = ts.wait(s4, before)) return rc;     // it wrote the same columns
        SplitGemm sg{};
        sg.A_planes = sg.B_planes = planes;
        sg.ldc = ld; sg.alpha = -1.f; sg.M = p0; sg.K = ow;
        if (split) {
            sg.a_panel0 = 0; sg.b_panel0 = (int)(p0 / 256); sg.C = H + p0;
            sg.N = OB;
            if (int rc = launch_gemm_split(sg, s4)) return rc;
        } else {
            Opt co; co.nk = true;
            if (int rc = gemm_on(s4, H + o0, ld, H + p0 * ld + o0, ld, H + p0, ld, p0, OB, ow, -1.f, co)) return rc;
        }
        if (int rc = ts.mark(s4, &strip_done)) return rc;
        if (int rc = ts.wait(s2, panel)) return rc;
        if (split) {
            sg.a_panel0 = sg.b_panel0 = 0; sg.C = H;
            sg.N = p0;
            sg.upper_square = true;
            if (int rc = launch_gemm_split(sg, s2)) return rc;
        } else {
            Opt ro; ro.nk = true; ro.upper = true;
            if (int rc = gemm_on(s2, H + o0, ld, H + o0, ld, H, ld, p0, p0, ow, -1.f, ro)) return rc;
        }
        if (int rc = ts.mark(s2, &rest_done)) return rc;
    }
    // everything back on the caller's stream
    for (hipStream_t st : {s2, s4, s3}) {
        hipEvent_t done = nullptr;
        if (int rc = ts.mark(st, &done)) return rc;
        if (int rc = ts.wait(s, done)) return rc;
    }

    // Nothing below the diagonal is part of the result (it holds the input's lower half and the below-diagonal parts of
    // straddling update tiles), and the triangular products of the inverse rely on zeros there.
    hipLaunchKernelGGL(zero_lower_kernel, dim3((unsigned)n), dim3(256), 0, s, H, ld, n);
    GPTQ_LAUNCH_CHECK();
    if (!want_inverse) return GPTQ_OK;

    // ---- U = R^-1 in place, right-looking over the outer block columns --------------------------------------------
    hipEvent_t panel_done = nullptr;     // s2: the last column panel, which reuses T
    hipEvent_t planes_free[2] = {};      // s2: the last product that reads the column planes
    for (int64_t k = 0; k < nouter; ++k) {
        const int64_t k0 = k * OB, k1 = std::min<int64_t>(k0 + OB, n), kw = k1 - k0;
        const float* Ukk = w.Uoo + k * (int64_t)OB * OB;
        unsigned char* const cp = column_planes[k & 1];
        hipEvent_t read_done = nullptr;  // s: the column block above k has been read by this step's update
        if (k0 > 0 && inverse_split) {
            // its pieces serve the update and the product with U_kk
            if (int rc = ts.wait(s, planes_free[k & 1])) return rc;
            if (int rc = launch_split_rows(H + k0, ld, k0, cp, s, kw)) return rc;
        }
        if (k0 > 0 && inverse_split && k1 < n) {
            if (int rc = ts.mark(s, &read_done)) return rc;
            if (int rc = launch_split_cols(H + k0 * ld + k1, ld, n - k1, w.planes2, s)) return rc;
            SplitGemm sg{};
            sg.A_planes = cp; sg.B_planes = w.planes2;
            sg.C = H + k1; sg.ldc = ld; sg.alpha = 1.f; sg.M = k0; sg.N = n - k1; sg.K = OB;
            if (int rc = launch_gemm_split(sg, s)) return rc;
        } else {
            if (k1 < n && k0 > 0) {
                // U[0:k0, k1:n] += U[0:k0, k] (-U_kk R[k, k1:n])   (U[0:k0, k] not yet multiplied by U_kk; the second factor is
                // what the factorisation left in the row block)
                Opt u;
                if (int rc = gemm_on(s, H + k0, ld, H + k0 * ld + k1, ld, H + k1, ld, k0, n - k1, kw, 1.f, u)) return rc;
            }
            if (int rc = ts.mark(s, &read_done)) return rc;
        }
        // On the other stream: U[0:k0, k] <- U[0:k0, k] U_kk, and the diagonal block.  Nothing later reads them.
        // The last column block has no update after it: it stays on the caller's stream (in float32 through the row-panel buffer, free
        // by now), beside the last but one on the other stream.
        const bool last = (k == nouter - 1) && nouter > 1;
        hipStream_t sp = last ? s : s2;
        if (k0 > 0 && inverse_split) {
            unsigned char* const up = last ? w.planes2 : diag_planes;
            if (int rc = launch_split_cols(Ukk, OB, kw, up, sp, kw)) return rc;
            if (!last) { if (int rc = ts.wait(s2, read_done)) return rc; }
            SplitGemm sg{};
            sg.A_planes = cp; sg.B_planes = up;
            sg.C = H + k0; sg.ldc = ld; sg.alpha = 1.f; sg.M = k0; sg.N = kw; sg.K = kw; sg.overwrite = true; sg.b_upper_tri = true;
            if (int rc = launch_gemm_split(sg, sp)) return rc;
            if (!last) { if (int rc = ts.mark(s2, &planes_free[k & 1])) return rc; }
        } else {
            if (!last) { if (int rc = ts.wait(s2, read_done)) return rc; }
            if (k0 > 0) {
                float* Tp = last ? w.T2 : w.T;
                Opt c; c.overwrite = true; c.btri = true;
                if (int rc = gemm_on(sp, H + k0, ld, Ukk, OB, Tp, OB, k0, kw, kw, 1.f, c)) return rc;
                if (int rc = copy2d(sp, H + k0, ld, Tp, OB, k0, kw)) return rc;
            }
        }
        hipLaunchKernelGGL(copy_block_kernel, dim3(256), dim3(256), 0, sp, H + k0 * ld + k0, ld, Ukk, (int64_t)OB, kw, (int)kw, 1);
        GPTQ_LAUNCH_CHECK();
        if (!last) { if (int rc = ts.mark(s2, &panel_done)) return rc; }
    }
    if (int rc = ts.wait(s, panel_done)) return rc;
    return GPTQ_OK;
}

extern "C" int gptq_damp_cholesky_inverse(float* H, int64_t ld, int64_t n, float percdamp,
                                          void* ws, size_t ws_bytes, int* info_dev, void* stream) {
    int rc;
    if (chol_check_args(H, ld, n, percdamp, info_dev, &rc)) return rc;
    if (!ws || !aligned(ws, 256) || ws_bytes < gptq_damp_cholesky_inverse_workspace_bytes(n))
        return fail(GPTQ_ERR_WORKSPACE, "damp_cholesky_inverse: workspace missing, misaligned or too small");
    return chol_run(H, ld, n, percdamp, ws, info_dev, static_cast<hipStream_t>(stream), true);
}

extern "C" size_t gptq_damp_cholesky_workspace_bytes(int64_t n) { return gptq_damp_cholesky_inverse_workspace_bytes(n); }

extern "C" int gptq_damp_cholesky(float* H, int64_t ld, int64_t n, float percdamp,
                                  void* ws, size_t ws_bytes, int* info_dev, void* stream) {
    int rc;
    if (chol_check_args(H, ld, n, percdamp, info_dev, &rc)) return rc;
    if (!ws || !aligned(ws, 256) || ws_bytes < gptq_damp_cholesky_workspace_bytes(n))
        return fail(GPTQ_ERR_WORKSPACE, "damp_cholesky: workspace missing, misaligned or too small");
    return chol_run(H, ld, n, percdamp, ws, info_dev, static_cast<hipStream_t>(stream), true, false);
}

// ---- the variant that allocates nothing -------------------------------------------------------------------
// Same kernels, their workspace in a library-owned device array of fixed size.  Each GPU holds its own copy of the
// array at its own address: the address is looked up once per device, with that device current, and only that
// pointer -- never the array's name, which in host code is a stand-in and no device address -- is handed to kernels.
namespace {
constexpr int64_t NOALLOC_MAX_N = GPTQ_NOALLOC_MAX_N;
constexpr size_t NOALLOC_BYTES = (size_t)(NOALLOC_MAX_N / NB) * NB * NB * sizeof(float)      // inverses of the 128 x 128 diagonal blocks
                                 + 3 * (size_t)NOALLOC_MAX_N * OB * sizeof(float)            // a column panel, a row panel, the U_oo blocks
                                 + 2 * TRIANGLE_WORDS * sizeof(float) + 2048;                // an outer block of R, packed twice
static __device__ __align__(256) unsigned char scratch[NOALLOC_BYTES];

constexpr int MAXDEV = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[MAXDEV] = {};

int scratch_for_current_device(void** out) {
    int dev = 0;
    GPTQ_HIP_CHECK(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAXDEV) return fail(GPTQ_ERR_UNSUPPORTED, "device ordinal %d out of range", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        GPTQ_HIP_CHECK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p || !aligned(p, 256)) return fail(GPTQ_ERR_HIP, "hipGetSymbolAddress gave an unusable address for the scratch array");
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return GPTQ_OK;
}
}  // namespace

extern "C" int64_t gptq_noalloc_max_n(void) { return NOALLOC_MAX_N; }

extern "C" int gptq_damp_cholesky_inverse_noalloc(float* H, int64_t ld, int64_t n, float percdamp, int* info_dev, void* stream) {
    int rc;
    if (chol_check_args(H, ld, n, percdamp, info_dev, &rc)) return rc;
    if (n > NOALLOC_MAX_N)
        return fail(GPTQ_ERR_UNSUPPORTED, "damp_cholesky_inverse_noalloc: n = %lld exceeds the %lld channels the library's static scratch "
                                          "array holds; use gptq_damp_cholesky_inverse with a caller workspace",
                    (long long)n, (long long)NOALLOC_MAX_N);
    static_assert(NOALLOC_MAX_N % OB == 0, "layout below assumes whole outer blocks");
    if (chol_ws_layout(nullptr, n, false).total > NOALLOC_BYTES) return fail(GPTQ_ERR_UNSUPPORTED, "damp_cholesky_inverse_noalloc: scratch layout exceeds the static array");
    void* ws = nullptr;
    if ((rc = scratch_for_current_device(&ws))) return rc;
    return chol_run(H, ld, n, percdamp, ws, info_dev, static_cast<hipStream_t>(stream), false, true, false);
}

extern "C" int gptq_check_info(const int* info_dev, int* host_info, void* stream) {
    if (!info_dev) return fail(GPTQ_ERR_INVALID_ARG, "check_info: info_dev is null");
    hipStream_t s = static_cast<hipStream_t>(stream);
    int v = 0;
    GPTQ_HIP_CHECK(hipMemcpyAsync(&v, info_dev, sizeof(int), hipMemcpyDeviceToHost, s));
    GPTQ_HIP_CHECK(hipStreamSynchronize(s));
    if (host_info) *host_info = v;
    if (v < 0) return fail(GPTQ_ERR_HIP, "the factorisation did not finish on the device: workgroups that wait for one another gave up; nothing is said about the matrix");
    if (v != 0) return fail(GPTQ_ERR_NOT_POSDEF, "pivot of column %d (1-based) was not positive", v);
    return GPTQ_OK;
}
