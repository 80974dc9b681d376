// Shared host-side helpers of the GPTQ gfx950 library: status codes, error text, launch checks.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdarg>
#include <initializer_list>
#include <cstdint>
#include <cstdio>

#include "../../include/gptq.h"

namespace gptq {

void set_error(const char* fmt, ...);

inline int fail(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
int fail_v(int code, const char* fmt, va_list ap);
inline int fail(int code, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    int rc = fail_v(code, fmt, ap);
    va_end(ap);
    return rc;
}

#define GPTQ_HIP_CHECK(expr)                                                                      \
    do {                                                                                          \
        hipError_t _e = (expr);                                                                   \
        if (_e != hipSuccess)                                                                     \
            return ::gptq::fail(GPTQ_ERR_HIP, "%s failed: %s", #expr, hipGetErrorString(_e));     \
    } while (0)

#define GPTQ_LAUNCH_CHECK() GPTQ_HIP_CHECK(hipGetLastError())

inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }
inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline size_t round_up(size_t a, size_t b) { return (a + b - 1) / b * b; }

// ---- look-ahead: helper streams and a ring of events (runtime.hip) ----------------------------
// The blocked solvers put the short, serial kernels of the next block column and the long trailing GEMM
// of the current one on different streams so that they overlap.  The helper streams (default priority,
// non-blocking) and their events are created once per host thread and device and live until the process
// ends.  Every use forks from and joins back into the caller's stream with events, so after an entry
// point returns all of its work is ordered on the caller's stream alone.
struct Lookahead {
    static constexpr int STREAMS = 3;
    hipStream_t streams[STREAMS] = {};
    hipEvent_t ev[32] = {};
    unsigned next = 0;
    hipEvent_t event() { return ev[next++ & 31]; }
};
int lookahead_get(Lookahead** out);     // for the current device; GPTQ_OK or an error code

// The streams of one entry point.  open(s, k) forks onto k of the library's helper streams; open(s, 0) keeps
// everything on the caller's stream (every side stream == main, no events: the same kernels in an order that respects
// every dependence, without overlap) -- for callers that must not create streams or events, and for calls that have nothing to
// put beside one another.  The destructor joins the helper streams back into the caller's on EVERY return path, so also after a
// launch failed half way through a call nothing is left running unordered beside the caller's stream.  An event of the ring
// may be recorded again while an earlier wait on it is still pending: a wait refers to the record that was current when it was
// enqueued.
struct HelperStreams {
    hipStream_t main = nullptr, side[Lookahead::STREAMS] = {};
    int helpers = 0;
    Lookahead* la = nullptr;
    int open(hipStream_t s, int count) {
        main = s;
        for (hipStream_t& st : side) st = s;
        if (count == 0) return GPTQ_OK;
        if (int rc = lookahead_get(&la)) return rc;
        // fork: nothing on a helper stream may start before the work already on the caller's stream (a helper's first
        // kernel may touch memory -- a workspace, say -- that earlier work of the caller still writes)
        hipEvent_t fork = la->event();
        GPTQ_HIP_CHECK(hipEventRecord(fork, main));
        for (; helpers < count; ++helpers) {
            side[helpers] = la->streams[helpers];
            GPTQ_HIP_CHECK(hipStreamWaitEvent(side[helpers], fork, 0));
        }
        return GPTQ_OK;
    }
    // *ev = a point on `on` that wait() can order another stream behind; stays null in single-stream mode
    int mark(hipStream_t on, hipEvent_t* ev) {
        *ev = nullptr;
        if (!la) return GPTQ_OK;
        hipEvent_t e = la->event();
        GPTQ_HIP_CHECK(hipEventRecord(e, on));
        *ev = e;
        return GPTQ_OK;
    }
    int wait(hipStream_t who, hipEvent_t ev) {
        if (!la || !ev) return GPTQ_OK;
        GPTQ_HIP_CHECK(hipStreamWaitEvent(who, ev, 0));
        return GPTQ_OK;
    }
    ~HelperStreams() {
        for (int i = 0; i < helpers; ++i) {
            hipEvent_t e = la->event();
            if (hipEventRecord(e, side[i]) == hipSuccess) (void)hipStreamWaitEvent(main, e, 0);
        }
    }
};

// ---- float32 matrix-core GEMM used by several steps (gemm_f32.hip) --------------------------
// C[M x N] += alpha * A[M x K] * op(B), A row-major (K contiguous).
//   b_is_nk = true : B is [N x K] row-major (K contiguous)  -> C += alpha * A * B^T
//   b_is_nk = false: B is [K x N] row-major (N contiguous)  -> C += alpha * A * B
//   overwrite: C = alpha * A * op(B) instead of accumulating.
//   upper_only: skip 128x128 output tiles that lie entirely below the diagonal (row0 > col0 + 127),
//               with (crow0, ccol0) the global offset of C's first element inside its parent matrix.
//   a_upper_tri: A[M x K] is the top-left part of an upper-triangular matrix (A[i][k] == 0 for k < i
//               rounded down to 128): the K loop of a tile starts at the tile's first row.
//   b_upper_tri: B given as [K x N] is the top-left part of an upper-triangular matrix with explicit zeros
//               below the diagonal: the K loop of a tile may end at the tile's last column (the large-tile
//               kernels do that; where it is not done the zeros give the same result).
// All pointers 16-byte aligned, leading dimensions multiples of 4.
struct GemmF32 {
    const float* A; int64_t lda;
    const float* B; int64_t ldb;
    float* C; int64_t ldc;
    int64_t M, N, K;
    float alpha;
    bool b_is_nk;
    bool overwrite;
    bool upper_only;
    int64_t crow0, ccol0;
    bool a_upper_tri;   // A is upper triangular with zeros below its diagonal blocks: skip k < first row of the tile
    bool b_upper_tri;   // B [K x N] is upper triangular with zeros below the diagonal: skip k > last column of the tile
};
int launch_gemm_f32(const GemmF32& g, hipStream_t s);

// ---- float32 products of rank 1024 on the bf16 matrix cores (gemm_split.hip) -----------------
// C[M x N] += alpha * A * B^T over K <= SPLIT_K, with both operands given as "planes": the three bfloat16 pieces of every
// float32 element in the blocked layout the kernel copies straight into LDS.
//   launch_split_rows: A [rows x k] float32, K contiguous        -> planes of ceil(rows / 256) panels
//   launch_split_cols: B [k x cols] float32, columns contiguous  -> planes of ceil(cols / 256) panels (of B^T)
// Both write into split_planes_bytes(rows) bytes; rows past the operand's end are zeros.  A launch reads panels a_panel0 .. and
// b_panel0 .. of the two plane buffers.
//   upper_square: C is square and only the 128 x 128 tiles of its upper triangle are computed (diagonal tiles whole).
// The six piece products kept leave a relative error of at most 2^-23 per product of two elements.
constexpr int SPLIT_K = 1024;
struct SplitGemm {
    const unsigned char* A_planes; int a_panel0;
    const unsigned char* B_planes; int b_panel0;
    float* C; int64_t ldc;
    float alpha;
    int64_t M, N, K;                    // M whole tiles of 128
    bool upper_square;
    bool whole_diagonal;                // ... of the 256 x 256 tiles that touch it, all four
    bool overwrite;                     // C = alpha * A * B^T instead of accumulating (C may be what A's planes were made from)
    bool b_upper_tri;                   // B^T [K x N] is upper triangular with zeros below the diagonal: skip k > last column of a tile
};
size_t split_planes_bytes(int64_t rows);
bool split_pays(int64_t tiles, bool otherwise);     // whether a launch of that many 256 x 256 tiles takes the split kernel (`otherwise`: unless a minimum is set)
int launch_split_rows(const float* A, int64_t lda, int64_t rows, unsigned char* planes, hipStream_t s, int64_t k = SPLIT_K);
int launch_split_cols(const float* B, int64_t ldb, int64_t cols, unsigned char* planes, hipStream_t s, int64_t k = SPLIT_K);
int launch_gemm_split(const SplitGemm& g, hipStream_t s);

}  // namespace gptq
