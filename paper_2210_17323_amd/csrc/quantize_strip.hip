// Step 3, the columns of one outer block (Algorithm 1, Section 3 Steps 1-3): a workgroup takes a strip of weight rows
// through all the blocks of 128 columns of an outer block of up to 1024 columns in ONE launch.  Rows are independent in
// Alg. 1 (the Hessian information is shared by all rows), so nothing crosses workgroups.
//
//   * The strip's working values -- RT * 16 rows x 1024 columns -- live in registers, as accumulators of v_mfma_f32_16x16x4_f32 that
//     hold the strip transposed: a lane is a weight row, its registers are columns.  Eight wavefronts, the updaters, own 16 columns of
//     every block of 128 still to come.
//   * A block is walked by one wavefront per 16 rows, a walker.  Its four DPP rows share the columns of those 16 rows; the four
//     columns of a quad lie in the four registers of one DPP row, which walks them -- grid value, error, update of the
//     quad's later columns --; then the quad's errors, spread over the four DPP rows as an operand, go into the later columns by matrix
//     instructions: into the next quad's tile at once, into the others between the steps of the next quad.
//   * Meanwhile the updaters apply the errors of the block before to the blocks after this one, and this block's, 16 columns
//     at a time as they are walked, to the next block.  That one is complete when its walk may begin but for the last 16 columns' products;
//     it goes to the walkers through LDS in the layout they take it in.
//
// What bounds it: a column is ~28 instructions of one wavefront (its chain, a quarter of the quad's overhead, and its matrix instructions,
// which on this chip take the vector units' cycles: 40 each), 9.9 us a block; with more rows a CU's vector units, which walkers
// and updaters share.  An outer block takes 95 / 136 / 191 us with 16 / 32 / 48 rows per workgroup (driven by R; strip_row_tiles has all
// forms).  With updates and walk one behind the other and a multiply-add per lane and column in the walk it took 144 / 181 / 232: Alg. 1 on a
// 4096 x 4096 layer 1.07 -> 0.84 ms, 3000 x 5120 in groups of 1024 1.48 -> 1.17 ms, 14336 x 14336 in groups of 128 20.9 -> 20.2 ms.
#include "quantize_common.h"
#include "split_planes.h"

#include <utility>

namespace gptq {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

namespace {

constexpr int NQ = QB / 4;              // quads of columns in a block
constexpr int NT = QB / 16;             // 16-column tiles of a block
constexpr int PW = QB + 4;              // pitch of the row buffers: 16 rows start on 16 different bank quads
constexpr int STRIP_BLOCKS = 8;         // blocks of an outer block
constexpr int PAIRS = STRIP_BLOCKS * (STRIP_BLOCKS - 1) / 2;
constexpr int UPDATERS = NT;            // wavefronts that hold the later blocks, 16 columns of each
// A block's triangular matrix, as it lies in LDS and (packed once per call) in the workspace: for every quad q of columns and every
// tile t from the quad's own on the operand that takes the quad's errors to the tile -- lane (l16, kq): M[4 q + kq][16 t + l16], zero up
// to the quad's last column --, then for every quad the values its own walk needs, 16 floats:
// M01 M02 M03 M12, M13 M23 - -, the diagonal M00 M11 M22 M33, and the hardware's reciprocal estimates of the diagonal.
constexpr int quad_words(int q) { return 64 * (4 * ((q >> 2) * NT - (q >> 2) * ((q >> 2) - 1) / 2) + (q & 3) * (NT - (q >> 2))); }      // words before quad q
constexpr int DIAG_FAR = quad_words(NQ);
constexpr int DIAG_WORDS = DIAG_FAR + NQ * 16;
constexpr int PAIR_WORDS = QB * QB;
static_assert(STRIP_DIAG_BYTES == DIAG_WORDS * 4 && STRIP_PAIR_BYTES == (size_t)PAIRS * PAIR_WORDS * 4, "quantize_common.h states these sizes");
static_assert(DIAG_WORDS % 256 == 0, "copied 1 KB at a time");

typedef __attribute__((address_space(3))) float* lds_float;
typedef const volatile __attribute__((address_space(3))) float* lds_float_ordered;
typedef const volatile __attribute__((address_space(3))) floatx2* lds_float2_ordered;
typedef const volatile __attribute__((address_space(3))) floatx4* lds_float4_ordered;

enum { FORM_U = 0, FORM_R = 1, FORM_HYBRID = 2 };

// A row's grid, ready for the decision  code = clamp(rint(x / scale) + zero, 0, maxq).
//   x / scale is the rounded quotient: scale = sn * 2^-es with sn in [0.5, 1), rs = 1 / sn, one correction step with the exact
//   remainder.  The estimate is held within FAR, far outside every code, so that an infinite quotient meets a finite product in the
//   remainder and keeps its sign; what is NaN takes code 0 (a median with NaN is the smallest of the others).
//   rint is the rounding of an addition: a float in [2^23, 2^24) has no fraction bits, and MAGIC is even, so ties go to
//   the even quotient.  Clamped there, between MAGIC - zero and MAGIC - zero + maxq (what lies outside the binade is
//   outside these bounds on the same side), the sum's low byte is OFF + code - zero: MAGIC is OFF past a multiple of 256.
//   zero is at most 22: -lo / scale exceeds maxq only where the scale is a denormal of few bits, 1.5 times at most.  Where the
//   range is so small that the scale itself is 0, every quotient is infinite, or NaN for a weight of 0: the zero point
//   (2^31 - 1) is stored but shifts nothing.
constexpr int OFF = 64;
constexpr float MAGIC = 12582912.f + (float)OFF;
constexpr float FAR = 1073741824.f;
struct RowGrid {
    float scale, sn, rs, lo, hi;
    int es, zero;
    uint32_t bias;                      // what four packed low bytes exceed the four codes by
    __device__ __forceinline__ void set(float s, int z, float maxq) {
        scale = s;
        zero = z;
        const bool finite = s < INFINITY, none = s == 0.f;   // an infinite scale (infinite weights): every quotient is 0 or NaN
        es = none ? 300 : (finite ? -__builtin_amdgcn_frexp_expf(s) : 0);
        sn = none || !finite ? 1.f : __builtin_amdgcn_frexp_mantf(s);
        float r = __builtin_amdgcn_rcpf(sn);
        r = fmaf(fmaf(-sn, r, 1.f), r, r);
        rs = finite ? r : (s == INFINITY ? 0.f : s);          // NaN stays NaN
        const int shift = none ? 0 : z;
        lo = MAGIC - (float)shift;
        hi = lo + maxq;
        bias = (uint32_t)(OFF - shift) * 0x01010101u;
    }
    // the clamped, rounded quotient of x, as MAGIC + (code - zero)
    __device__ __forceinline__ float decide(float x) const {
        const float xs = ldexpf(x, es);
        const float x0 = __builtin_amdgcn_fmed3f(xs * rs, -FAR, FAR);
        return __builtin_amdgcn_fmed3f(fmaf(fmaf(-x0, sn, xs), rs, x0) + MAGIC, lo, hi);
    }
};

// The walk of one block by one wavefront.
template <int FORM>
struct Walk {
    floatx4 w[NT];                      // this lane's row, columns 16 t + 4 kq + e
    floatx4 n0[2], nd[2], nr[2];        // M01 M02 M03 M12, the diagonal and its reciprocals (this quad, next quad)
    floatx2 n1[2];                      // M13 M23
    floatx4 orig[2];                    // original weights of the quad's columns (R and hybrid forms)
    float far[3][NT];                   // the operands that take a quad's errors to the tiles (the quad before, this one, the next)
    float spread;                       // the errors of the quad before, as an operand
    RowGrid grid;
    float maxq, e2;
    int kq;
    lds_float lane_diag;                // block matrix + lane
    lds_float diag;
    lds_float orow;                     // this row of the original weights
    lds_float erow;                     // this row of the strip's error block
    uint32_t __attribute__((address_space(3)))* crow;      // this row's codes, four to a word
};

template <int I, int FORM>
__device__ __forceinline__ void request_quad(Walk<FORM>& s) {
    if constexpr (I < NQ) {
        s.n0[I & 1] = *(lds_float4_ordered)(s.diag + DIAG_FAR + 16 * I);
        s.nd[I & 1] = *(lds_float4_ordered)(s.diag + DIAG_FAR + 16 * I + 8);
        s.nr[I & 1] = *(lds_float4_ordered)(s.diag + DIAG_FAR + 16 * I + 12);
        s.n1[I & 1] = *(lds_float2_ordered)(s.diag + DIAG_FAR + 16 * I + 4);
        if constexpr (FORM != FORM_U) s.orig[I & 1] = *(lds_float4_ordered)(s.orow + 4 * I);
#pragma unroll
        for (int t = I / 4; t < NT; ++t) s.far[I % 3][t] = *(lds_float_ordered)(s.lane_diag + quad_words(I) + 64 * (t - I / 4));
    }
}

struct Pair { float a, b; };
__device__ __forceinline__ Pair swap16(float a, float b) {      // {a0 b0 a2 b2}, {a1 b1 a3 b3} of the DPP rows
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ Pair swap32(float a, float b) {      // {a0 a1 b0 b1}, {a2 a3 b2 b3}
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}
// DPP row c of the result: v[c] of DPP row ROW
template <int ROW>
__device__ __forceinline__ float spread_row(const float (&v)[4]) {
    const Pair p = swap16(v[0], v[1]), q = swap16(v[2], v[3]);
    const Pair r = (ROW & 1) ? swap32(p.b, q.b) : swap32(p.a, q.a);
    return ROW < 2 ? r.a : r.b;
}
// the smallest / largest of the DPP rows FIRST .. FIRST + COUNT - 1 (COUNT 2 or 4), in every DPP row
template <int FIRST, int COUNT, class F>
__device__ __forceinline__ float across_rows(float v, F f) {
    const Pair h = swap32(v, v);                         // {0 1 0 1}, {2 3 2 3}
    if constexpr (COUNT == 4) {
        const float m = f(h.a, h.b);
        const Pair p = swap16(m, m);
        return f(p.a, p.b);
    } else {
        const float m = FIRST == 0 ? h.a : h.b;
        const Pair p = swap16(m, m);
        return f(p.a, p.b);
    }
}

// Grid of the group of COLS columns that starts at quad I, from the weights as they stand
template <int I, int COLS, int FORM>
__device__ __forceinline__ void group_grid(Walk<FORM>& s, int grid) {
    float lo = s.w[I / 4][0], hi = lo;
#pragma unroll
    for (int t = 0; t < (COLS + 15) / 16; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) { lo = fminf(lo, s.w[I / 4 + t][e]); hi = fmaxf(hi, s.w[I / 4 + t][e]); }
    constexpr int COUNT = COLS == 8 ? 2 : 4;
    lo = across_rows<I & 3, COUNT>(lo, [](float a, float b) { return fminf(a, b); });
    hi = across_rows<I & 3, COUNT>(hi, [](float a, float b) { return fmaxf(a, b); });
    float sc; int zr;
    grid_from_range(grid, s.maxq, lo, hi, fmaxf(fabsf(lo), fabsf(hi)), sc, zr);
    s.grid.set(sc, zr, s.maxq);
}

struct GroupOut { float* scales; int32_t* zeros; };        // this row's first group of the block

// Before the quads where a group of 32 columns or more may start, every column has to be as it stands.
constexpr bool flushed(int form, int quad) { return form != FORM_R && quad % 8 == 0; }

// One quad of columns.  Its four columns lie in the four registers of DPP row I % 4 of tile I / 4; the other lanes go through the same
// motions on columns that are not due yet, and nothing of that is kept.
template <int I, int FORM>
__device__ __forceinline__ void walk_quad(Walk<FORM>& s, int in_group, int kind, int nbk, const GroupOut& go) {
    constexpr int T = I / 4, ROW = I & 3;
    // what the quad before left: its errors into the tiles behind this one's, two a column, where the chain leaves the issue slots
    // free (behind one another each would hold the wavefront for the 32 cycles that the one before takes)
    constexpr int LEFT = I > 0 && !flushed(FORM, I) ? NT - 1 - T : 0;
    request_quad<I + 1, FORM>(s);
    if constexpr (FORM != FORM_R) {
        // a group starts here (in_group: columns of a group inside the block, 0 otherwise; the same for all lanes)
        bool start = false;
        if constexpr (I % 2 == 0) { if (in_group == 8) { group_grid<I, 8>(s, kind); start = true; } }
        if constexpr (I % 4 == 0) { if (in_group == 16) { group_grid<I, 16>(s, kind); start = true; } }
        if constexpr (I % 8 == 0) { if (in_group == 32) { group_grid<I, 32>(s, kind); start = true; } }
        if constexpr (I % 16 == 0) { if (in_group == 64) { group_grid<I, 64>(s, kind); start = true; } }
        if constexpr (I == 0) { if (in_group == 128) { group_grid<I, 128>(s, kind); start = true; } }
        if constexpr (I % 2 == 0) {
            if (start && 4 * I < nbk && s.kq == 0 && go.scales) {
                const int gi = (4 * I) / in_group;
                go.scales[gi] = s.grid.scale;
                go.zeros[gi] = s.grid.zero;
            }
        }
    }
    float x[4] = {s.w[T][0], s.w[T][1], s.w[T][2], s.w[T][3]};
    float t[4], ne[4], e[4];
    floatx4 out;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        const float mjj = s.nd[I & 1][a], rcp = s.nr[I & 1][a];
        if constexpr (FORM == FORM_R) {
            // the weight Alg. 1 holds here is w_j + s_j / R_jj: reciprocal estimate and one correction step with the exact
            // remainder (R_jj is the square root of a pivot of the damped Hessian: no range scaling needed)
            const float t0 = x[a] * rcp;
            const float wj = s.orig[I & 1][a];
            const float wn = wj + fmaf(fmaf(-t0, mjj, x[a]), rcp, t0);
            t[a] = s.grid.decide(wn);
            const float cz = t[a] - MAGIC;                                  // code - zero; the grid value is scale * cz
            ne[a] = fmaf(-s.grid.scale, cz, wj);                            // d_j
            e[a] = fmaf(-s.grid.scale, cz, wn) * mjj;
            out[a] = ne[a];
        } else {
            t[a] = s.grid.decide(x[a]);
            const float cz = t[a] - MAGIC;
            // e = (w - q) / U_jj in the same way
            const float d = fmaf(s.grid.scale, cz, -x[a]);                  // q - w
            const float e0 = d * rcp;
            e[a] = ne[a] = fmaf(fmaf(-e0, mjj, d), rcp, e0);                // -e: only its square is wanted besides
            out[a] = FORM == FORM_U ? ne[a] : fmaf(-s.grid.scale, cz, s.orig[I & 1][a]);
        }
#pragma unroll
        for (int u = 2 * a; u < 2 * a + 2; ++u)
            if (u < LEFT) s.w[T + 1 + u] = __builtin_amdgcn_mfma_f32_16x16x4f32(s.far[(I + 2) % 3][T + 1 + u], s.spread, s.w[T + 1 + u], 0, 0, 0);
        if (a == 0) { x[1] = fmaf(ne[0], s.n0[I & 1][0], x[1]); x[2] = fmaf(ne[0], s.n0[I & 1][1], x[2]); x[3] = fmaf(ne[0], s.n0[I & 1][2], x[3]); }
        if (a == 1) { x[2] = fmaf(ne[1], s.n0[I & 1][3], x[2]); x[3] = fmaf(ne[1], s.n1[I & 1][0], x[3]); }
        if (a == 2) x[3] = fmaf(ne[2], s.n1[I & 1][1], x[3]);
#pragma unroll
        for (int u = 0; u < 2; ++u)
            if (2 * a + u < LEFT) {
                __builtin_amdgcn_sched_group_barrier(0x002, 9, 0);       // vector instructions
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);       // a matrix instruction
            }
        __builtin_amdgcn_sched_barrier(0);
    }
    // the quad's errors to the next quad's tile, at once
    if constexpr (I + 1 < NQ) {
        s.spread = spread_row<ROW>(ne);
        constexpr int FIRST = (I + 1) / 4;
        s.w[FIRST] = __builtin_amdgcn_mfma_f32_16x16x4f32(s.far[I % 3][FIRST], s.spread, s.w[FIRST], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (flushed(FORM, I + 1)) {
#pragma unroll
            for (int u = FIRST + 1; u < NT; ++u) s.w[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(s.far[I % 3][u], s.spread, s.w[u], 0, 0, 0);
        }
    }
    // the four low bytes, side by side
    const uint32_t c01 = __builtin_amdgcn_perm(__float_as_uint(t[1]), __float_as_uint(t[0]), 0x0c0c0400u);
    const uint32_t c23 = __builtin_amdgcn_perm(__float_as_uint(t[3]), __float_as_uint(t[2]), 0x04000c0cu);
    const uint32_t code = (c01 | c23) - s.grid.bias;
    if (s.kq == ROW) {
#pragma unroll
        for (int a = 0; a < 4; ++a) s.e2 = fmaf(e[a], e[a], s.e2);
        *(__attribute__((address_space(3))) floatx4*)(s.erow + 4 * I) = out;
        s.crow[I] = code;
    }
    __builtin_amdgcn_sched_barrier(0);
}

template <int FORM, int FIRST, int... I>
__device__ __forceinline__ void walk_quads(Walk<FORM>& s, int in_group, int kind, int nbk, const GroupOut& go, std::integer_sequence<int, I...>) {
    (walk_quad<FIRST + I, FORM>(s, in_group, kind, nbk, go), ...);
}

__device__ __forceinline__ float weight_at(const void* W, int wdtype, int64_t i) {
    if (wdtype == GPTQ_F16) return (float)static_cast<const _Float16*>(W)[i];
    if (wdtype == GPTQ_BF16) return (float)static_cast<const __bf16*>(W)[i];
    return static_cast<const float*>(W)[i];
}

// four weights as they lie in memory (16-bit types: in the first two words)
__device__ __forceinline__ floatx4 as_weights(floatx4 raw, int wdtype) {
    if (wdtype == GPTQ_F32) return raw;
    const uint32_t x = __float_as_uint(raw[0]), y = __float_as_uint(raw[1]);
    if (wdtype == GPTQ_BF16) return floatx4{__uint_as_float(x << 16), __uint_as_float(x & 0xffff0000u), __uint_as_float(y << 16), __uint_as_float(y & 0xffff0000u)};
    return floatx4{(float)__builtin_bit_cast(_Float16, (uint16_t)x), (float)__builtin_bit_cast(_Float16, (uint16_t)(x >> 16)),
                   (float)__builtin_bit_cast(_Float16, (uint16_t)y), (float)__builtin_bit_cast(_Float16, (uint16_t)(y >> 16))};
}

// STRIP_PACK_OUTER outer blocks of the factor, from column j_first on, as the strip kernel reads them.  DIAG_PARTS workgroups for every one
// of nblk diagonal blocks (identity outside the matrix), then two per 128 x 128 tile above the diagonal blocks of an outer block (64 rows each), in the
// order in which the lanes take operands: [wavefront: 16 columns][16 rows][lane: column][4 rows], zeros outside the matrix.  Read as it lies, 128 columns of a factor whose rows are a multiple of 4 KB apart come from two of an
// XCD's sixteen L2 channels, with every CU of the chip reading the same 512 bytes of each row at the same time.
constexpr int DIAG_PARTS = 16;

__global__ __launch_bounds__(256) void pack_factor_kernel(const float* M, int64_t ldm, const float* D, int64_t ldd, int diag_dense,
                                                          int64_t n, int64_t j_first, int nblk, float* diag_out, float* pair_out) {
    __shared__ float tile[64][QB + 1];
    const int tid = threadIdx.x;
    // (with one workgroup a block its 64 short loads behind one another were what the launch waited for, 19 us whatever the size)
    if ((int)blockIdx.x < nblk * DIAG_PARTS) {
        const int blk = (int)blockIdx.x / DIAG_PARTS, part = (int)blockIdx.x % DIAG_PARTS;
        const int64_t j0 = j_first + (int64_t)blk * QB;
        const float* B = D + (diag_dense ? j0 * QB : j0 * ldd + j0);
        const int64_t ld = diag_dense ? QB : ldd;
        const int lim = diag_dense ? QB : (int)min((int64_t)QB, n - j0);
        float* out = diag_out + (int64_t)blk * DIAG_WORDS;
        auto at = [&](int j, int k) { return (j < lim && k < lim) ? B[j * ld + k] : (j == k ? 1.f : 0.f); };
        for (int f = 4 * part + (tid >> 6); f < NQ * NT; f += 4 * DIAG_PARTS) {
            const int q = f / NT, t = f % NT, j = 4 * q + ((tid >> 4) & 3), k = 16 * t + (tid & 15);
            if (t < q / 4) continue;
            out[quad_words(q) + 64 * (t - q / 4) + (tid & 63)] = k > 4 * q + 3 ? at(j, k) : 0.f;
        }
        for (int q = part * 256 + tid; q < NQ * 16; q += 256 * DIAG_PARTS) {
            const int c = 4 * (q >> 4), e = q & 15;
            float v = 0.f;
            if (e < 3) v = at(c, c + 1 + e);
            else if (e < 5) v = at(c + 1, c + e - 1);
            else if (e == 5) v = at(c + 2, c + 3);
            else if (e >= 12) v = __builtin_amdgcn_rcpf(at(c + e - 12, c + e - 12));
            else if (e >= 8) v = at(c + e - 8, c + e - 8);
            out[DIAG_FAR + q] = v;
        }
        return;
    }
    const int rest = (int)blockIdx.x - nblk * DIAG_PARTS, p = rest >> 1, h = rest & 1;
    const int o = p / PAIRS;
    int q = p - o * PAIRS, b = 0;
    for (int left = STRIP_BLOCKS - 1; q >= left; --left) { q -= left; ++b; }
    const int64_t k0 = j_first + ((int64_t)o * STRIP_BLOCKS + b) * QB, c0 = k0 + (int64_t)(q + 1) * QB;
    if (c0 >= n) return;                                    // then the tile's rows are all inside the matrix
    for (int i = tid; i < 64 * 32; i += 256) {
        const int rr = i >> 5, cc = (i & 31) * 4;
        const float* src = M + (k0 + 64 * h + rr) * ldm + c0 + cc;
        floatx4 v = {0.f, 0.f, 0.f, 0.f};
        if (c0 + cc + 4 <= n) v = *reinterpret_cast<const floatx4*>(src);
        else {
#pragma unroll
            for (int e = 0; e < 4; ++e) if (c0 + cc + e < n) v[e] = src[e];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) tile[rr][cc + e] = v[e];
    }
    __syncthreads();
    float* out = pair_out + (int64_t)p * PAIR_WORDS;
    for (int i = tid; i < 64 * 32; i += 256) {              // 16-byte pieces of this half: [wavefront][4 row groups][lane]
        const int lane = i & 63, t = (i >> 6) & 3, u = i >> 8;
        const int col = 16 * u + (lane & 15), k = 16 * t + 4 * (lane >> 4);
        const floatx4 v = {tile[k][col], tile[k + 1][col], tile[k + 2][col], tile[k + 3][col]};
        *reinterpret_cast<floatx4*>(out + ((u * 8 + 4 * h + t) * 64 + lane) * 4) = v;
    }
}

// No memory access moves across, for the compiler: between a count in LDS and the data that it stands for.  (The hardware takes a
// wavefront's LDS accesses in order, so it costs no instruction.)
__device__ __forceinline__ void compiler_fence() { asm volatile("" ::: "memory"); }

// A barrier that orders LDS accesses only: __syncthreads() would also wait for every global access in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// The wavefronts of a workgroup go to the SIMDs in turn.  Walkers are the first RT, a SIMD each; of the others those stay idle (bits of
// IDLE) that would share a walker's SIMD: beside one updater fewer a walker waits less for the matrix core.
constexpr int STRIP_WAVES = 12;
template <int RT> constexpr uint32_t IDLE = RT == 1 ? 0x910 : (RT == 2 ? 0x300 : 0x400);

template <int FORM, int RT>
__global__ __launch_bounds__(64 * STRIP_WAVES) void alg1_strip_kernel(StripArgs g) {
    constexpr int ROWS = 16 * RT;
    static_assert(STRIP_WAVES - RT - __builtin_popcount(IDLE<RT>) == UPDATERS, "eight wavefronts update");
    __shared__ __attribute__((aligned(16))) float diag[2][DIAG_WORDS];
    __shared__ __attribute__((aligned(16))) float ebuf[2][ROWS * PW];      // a block's working values, then its errors; blocks take turns
    __shared__ __attribute__((aligned(16))) float obuf[FORM == FORM_U ? 4 : ROWS * PW];     // the block's original weights
    __shared__ __attribute__((aligned(16))) uint32_t cbuf[ROWS * NQ];      // codes
    __shared__ int walked[RT];                                             // tiles, over all blocks
    __shared__ float red[2][UPDATERS][FORM == FORM_U ? ROWS : 1];          // group ranges of the updaters

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, kq = lane >> 4;
    const int64_t row0 = (int64_t)blockIdx.x * ROWS;
    const int nblocks = (int)((g.o1 - g.o0 + QB - 1) / QB);
    auto group_starts = [&](int b) { return FORM == FORM_U && g.wide_group && (g.o0 + (int64_t)b * QB) % g.wide_group == 0; };       // of several blocks

    if ((IDLE<RT> >> wave) & 1) return;
    // Barriers of a block: when its working values are in LDS, and behind its walk.  In between a walker counts its 16-column tiles, and
    // waits for nobody.
    if (wave < RT) {
        // ================ the walk: 16 rows per wavefront
        const int64_t wrow = row0 + 16 * wave + l16, wrow_c = min(wrow, g.r - 1);
        Walk<FORM> s;
        s.maxq = (float)g.maxq;
        s.grid.set(1.f, 0, s.maxq);
        s.kq = kq;
        double half = 0.0;
        if (g.in_group == 0 && g.wide_group == 0) {
            const int64_t gi = wrow_c * g.ngroups + (g.group ? g.o0 / g.group : 0);
            s.grid.set(g.scales[gi], g.zeros[gi], s.maxq);
        }
        if (g.half_e2 && g.o0 > 0) half = g.half_e2[wrow_c];
        const int rr = 16 * wave + l16;
        s.orow = FORM == FORM_U ? (lds_float)obuf : (lds_float)obuf + rr * PW;
        s.crow = (uint32_t __attribute__((address_space(3)))*)cbuf + rr * NQ;
#pragma unroll 1
        for (int b = 0; b < nblocks; ++b) {
            const int64_t j0 = g.o0 + (int64_t)b * QB;
            const int nbk = (int)min((int64_t)QB, g.n - j0);
            s.diag = (lds_float)diag + (b & 1) * DIAG_WORDS;
            s.lane_diag = s.diag + lane;
            s.erow = (lds_float)ebuf + ((b & 1) * ROWS + rr) * PW;
            lds_barrier();                              // the block is there
            if (group_starts(b)) {
                float lo = red[0][0][rr], hi = red[1][0][rr];
#pragma unroll
                for (int u = 1; u < UPDATERS; ++u) { lo = fminf(lo, red[0][u][rr]); hi = fmaxf(hi, red[1][u][rr]); }
                float sc; int zr;
                grid_from_range(g.grid, s.maxq, lo, hi, fmaxf(fabsf(lo), fabsf(hi)), sc, zr);
                s.grid.set(sc, zr, s.maxq);
                if (kq == 0 && wrow < g.r) {
                    g.scales[wrow * g.ngroups + j0 / g.wide_group] = sc;
                    g.zeros[wrow * g.ngroups + j0 / g.wide_group] = zr;
                }
            }
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                s.w[t] = *(__attribute__((address_space(3))) floatx4*)(s.erow + 16 * t + 4 * kq);
                if constexpr (FORM == FORM_HYBRID) s.w[t] += *(__attribute__((address_space(3))) floatx4*)(s.orow + 16 * t + 4 * kq);
            }
            s.e2 = 0.f;
            GroupOut go{nullptr, nullptr};
            if (g.in_group && wrow < g.r) {
                const int64_t gi = wrow * g.ngroups + j0 / g.in_group;
                go.scales = g.scales + gi;
                go.zeros = g.zeros + gi;
            }
            request_quad<0, FORM>(s);
            [&]<int... T>(std::integer_sequence<int, T...>) {
                ((walk_quads<FORM, 4 * T>(s, g.in_group, g.grid, nbk, go, std::make_integer_sequence<int, 4>{}),
                  compiler_fence(),
                  *(volatile __attribute__((address_space(3))) int*)(&walked[wave]) = NT * b + T + 1), ...);        // behind the tile's errors: LDS takes a wavefront's stores in order
            }(std::make_integer_sequence<int, NT>{});
            lds_barrier();
            // the row's sum: the columns of its four lanes
            {
                float v = s.e2;
                const Pair h = swap32(v, v);
                v = h.a + h.b;
                const Pair p = swap16(v, v);
                half += 0.5 * (double)(p.a + p.b);
            }
            // codes: 16 rows of 128, a row by 8 lanes
#pragma unroll
            for (int q = lane; q < 16 * 8; q += 64) {
                const int cr = 16 * wave + (q >> 3), k = (q & 7) * 16;
                if (row0 + cr >= g.r) continue;
                uint8_t* dst = g.codes + (row0 + cr) * g.ldc + j0 + k;
                const uint4 v = *reinterpret_cast<const uint4*>(&cbuf[cr * NQ + (k >> 2)]);
                if (k + 16 <= nbk && (reinterpret_cast<uintptr_t>(dst) & 15) == 0) {
                    *reinterpret_cast<uint4*>(dst) = v;
                } else {
                    const uint32_t wds[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int c = 0; c < 16; ++c)
                        if (k + c < nbk) dst[c] = (uint8_t)(wds[c >> 2] >> (8 * (c & 3)));
                }
            }
        }
        if (kq == 0 && wrow < g.r && g.half_e2) g.half_e2[wrow] = half;
        return;
    }

    // ================ the later blocks: wavefront u holds columns 16 u .. 16 u + 15 of each, transposed like the walkers' -- lane
    //                  (l16, kq): row 16 rt + l16, columns 4 kq + e of the tile.  Rows past r repeat the last one and are never stored;
    //                  columns past the outer block are zero.
    const int u = wave - RT - __builtin_popcount(IDLE<RT> & ((1u << wave) - 1)), utid = 64 * u + lane;
    floatx4 acc[STRIP_BLOCKS - 1][RT];                  // blocks b + 1 + j while block b is walked
    floatx4 head[RT];                                   // the block that is handed over next
    {
        const int wcol = 16 * u + 4 * kq;
        auto load_block = [&](int i, floatx4 (&d)[RT]) {
            const int64_t left = strip_block_columns(g.o0, g.o1, i);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                const float* p = g.S + min(row0 + 16 * rt + l16, g.r - 1) * g.lds_ + g.o0 + i * QB + wcol;
                d[rt] = floatx4{0.f, 0.f, 0.f, 0.f};
                if (!g.S || wcol >= left) continue;
                if (wcol + 4 <= left) d[rt] = *reinterpret_cast<const floatx4*>(p);
                else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) if (wcol + e < left) d[rt][e] = p[e];
                }
            }
        };
        load_block(0, head);
#pragma unroll
        for (int i = 1; i < STRIP_BLOCKS; ++i) load_block(i, acc[i - 1]);
    }
    auto load_diag = [&](int b) {                       // straight into LDS, 1 KB per wavefront and instruction
        const float* src = g.diag + (int64_t)b * DIAG_WORDS + lane * 4;
        float* dst = diag[b & 1];
        for (int t = u; t < DIAG_WORDS / 256; t += UPDATERS)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + 256 * t),
                                             (__attribute__((address_space(3))) void*)(dst + 256 * t), 16, 0, 0);
    };
    // The original weights are requested as they are and turned into float32 only when they are put into LDS, so that
    // nothing waits for them in between.  Rows that cannot be read four weights at a time are read there, one by one.
    floatx4 oreg[FORM == FORM_U ? 1 : RT];
    auto orig_whole = [&](int64_t j0) { return g.w_vec && j0 + QB <= g.n; };
    auto orig_at = [&](int64_t j0, int t) {
        const int q = utid + 64 * UPDATERS * t;
        return min(row0 + (q >> 5), g.r - 1) * g.ldw + j0 + (q & 31) * 4;
    };
    auto load_orig = [&](int64_t j0) {
        if constexpr (FORM != FORM_U) {
            if (!orig_whole(j0)) return;
            if (g.wdtype == GPTQ_F32) {
#pragma unroll
                for (int t = 0; t < RT; ++t) oreg[t] = *reinterpret_cast<const floatx4*>(static_cast<const float*>(g.W) + orig_at(j0, t));
            } else {
#pragma unroll
                for (int t = 0; t < RT; ++t) {
                    const floatx2 v = *reinterpret_cast<const floatx2*>(static_cast<const uint16_t*>(g.W) + orig_at(j0, t));
                    oreg[t][0] = v[0]; oreg[t][1] = v[1];
                }
            }
        }
    };
    auto store_orig = [&](int64_t j0) {
        if constexpr (FORM != FORM_U) {
            const bool whole = orig_whole(j0);
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                const int q = utid + 64 * UPDATERS * t, k = (q & 31) * 4;
                floatx4 v = {0.f, 0.f, 0.f, 0.f};
                if (whole) {
                    v = as_weights(oreg[t], g.wdtype);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const bool in = j0 + k + e < g.n;
                        const float x = weight_at(g.W, g.wdtype, orig_at(j0, t) + (in ? e : -k));       // a column past n reads the block's first
                        v[e] = in ? x : 0.f;
                    }
                }
                *reinterpret_cast<floatx4*>(&obuf[(q >> 5) * PW + k]) = v;
            }
        }
    };
    // block b, whose working values are in `head`, to the walkers
    auto hand_over = [&](int b) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) *reinterpret_cast<floatx4*>(&ebuf[b & 1][(16 * rt + l16) * PW + 16 * u + 4 * kq]) = head[rt];
        if (group_starts(b)) {                          // a group of several blocks: its range over the current values of all its columns
            const int gb = (int)(g.wide_group / QB);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                float lo = head[rt][0], hi = lo;
#pragma unroll
                for (int e = 1; e < 4; ++e) { lo = fminf(lo, head[rt][e]); hi = fmaxf(hi, head[rt][e]); }
#pragma unroll
                for (int j = 0; j < STRIP_BLOCKS - 1; ++j)
                    if (j + 1 < gb) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) { lo = fminf(lo, acc[j][rt][e]); hi = fmaxf(hi, acc[j][rt][e]); }
                    }
                lo = across_rows<0, 4>(lo, [](float a, float b) { return fminf(a, b); });
                hi = across_rows<0, 4>(hi, [](float a, float b) { return fmaxf(a, b); });
                if (kq == 0) { red[0][u][16 * rt + l16] = lo; red[1][u][16 * rt + l16] = hi; }
            }
        }
        store_orig(g.o0 + (int64_t)b * QB);
    };
    // The tile (b, b') of the packed factor, this wavefront's 16 columns of it, two groups of 16 k at a time (`part` 0 .. 3)
    // (as an offset that is the same for the wavefront: as addresses, one for every unit below, they would fill the registers)
    const auto pairs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(g.pairs), 0, (int)STRIP_PAIR_BYTES, 0x00020000);
    const int pair_lane = (u * 512 + lane) * 16;
    auto tile_part = [&](int b, int b2, int part) { return (b * (2 * STRIP_BLOCKS - 1 - b) / 2 + b2 - b - 1) * (PAIR_WORDS * 4) + part * 2048; };
    auto request = [&](int offset, floatx4 (&d)[2]) {
        d[0] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(pairs, pair_lane, offset, 0));
        d[1] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(pairs, pair_lane + 1024, offset, 0));
    };
    // d += (E_b columns 16 group .. 16 group + 15) (the tile's rows of these); E_b in LDS
    auto multiply_group = [&](int b, int group, floatx4 m, floatx4 (&d)[RT]) {
        floatx4 x[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) x[rt] = *reinterpret_cast<const floatx4*>(&ebuf[b & 1][(16 * rt + l16) * PW + 16 * group + 4 * kq]);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) d[rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(m[e], x[rt][e], d[rt], 0, 0, 0);
    };
    auto multiply = [&](int b, int part, const floatx4 (&m)[2], floatx4 (&d)[RT]) {
        multiply_group(b, 2 * part, m[0], d);
        multiply_group(b, 2 * part + 1, m[1], d);
    };
    // Block e's errors to the blocks from e + 2 on, `count` units (unit j is block e + 2 + j, held in acc[j + base]).  A block's 128 products are summed on their own and added once: one by one, each would be rounded at the size of the running value.
    constexpr int RING = RT == 1 ? 4 : 2;                // parts of tiles on their way or in use (two row tiles with four: 266 us for two rounds, with two 257)
    floatx4 ring[RING][2];
    auto start_units = [&](int e) {
#pragma unroll
        for (int q = 0; q < RING - 1; ++q) request(tile_part(e, min(e + 2, nblocks - 1), q), ring[q]);
    };
    auto units = [&](int e, auto BASE, int count) {
        constexpr int base = decltype(BASE)::value;
        const int end = nblocks - 1;                    // past the last tile the loads repeat it
#pragma unroll
        for (int j = 0; j + base < STRIP_BLOCKS - 1; ++j) {
            if (j >= count) break;
            floatx4 sum[RT];
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) sum[rt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int ahead = q + RING - 1;
                request(tile_part(e, min(e + 2 + j + ahead / 4, end), ahead % 4), ring[ahead % RING]);
                __builtin_amdgcn_sched_barrier(0);
                multiply(e, q, ring[q % RING], sum);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) acc[j + base][rt] += sum[rt];
        }
    };
    // a block's errors to memory, as they are or as the pieces that the update beyond the outer block multiplies
    auto write_errors = [&](int b) {
        if (!g.E && !g.E_planes) return;
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            const int q = utid + 64 * UPDATERS * t, rr = q >> 5, k = (q & 31) * 4;
            if (row0 + rr >= g.r) continue;
            const floatx4 e = *reinterpret_cast<const floatx4*>(&ebuf[b & 1][rr * PW + k]);
            if (g.E_planes) store_pieces(g.E_planes, row0 + rr, b * QB + k, make_float4(e[0], e[1], e[2], e[3]));
            else *reinterpret_cast<floatx4*>(g.E + (row0 + rr) * g.lde + b * QB + k) = e;
        }
    };
    if (u == 0 && lane < RT) walked[lane] = 0;
    load_diag(0);
    load_orig(g.o0);
    hand_over(0);
    __builtin_amdgcn_s_waitcnt(0x0F70);                 // vmcnt(0): the first block's matrix is in LDS
    bool behind = false;                                // block b - 1's errors are still to go to the blocks from b + 1 on
#pragma unroll 1
    for (int b = 0; b < nblocks; ++b) {
        const int64_t j0 = g.o0 + (int64_t)b * QB;
        const int later = nblocks - 1 - b;
        const int n_units = behind ? later : 0;         // block b - 1's errors: blocks b + 1 ..
        floatx4 near, sum[RT];                          // the tile (b, b + 1), 16 rows at a time, and this block's products into the next
        int taken = 0;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) sum[rt] = floatx4{0.f, 0.f, 0.f, 0.f};
        const int near_tile = tile_part(b, b + 1, 0);
        auto request_near = [&](int group) { near = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(pairs, pair_lane, near_tile + min(group, NT - 1) * 1024, 0)); };
        auto take = [&](int upto) {
#pragma unroll 1
            while (taken < upto) {
                multiply_group(b, taken, near, sum);
                request_near(++taken);
            }
        };
        auto walked_tiles = [&] {                       // of this block, by all walkers
            int v = NT;
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) v = min(v, *(volatile __attribute__((address_space(3))) int*)(&walked[rt]) - NT * b);
            v = __builtin_amdgcn_readfirstlane(v);
            compiler_fence();                           // the errors are read behind the count
            return v;
        };
        lds_barrier();                                  // the walk of block b starts
        if (later > 0) {
            request_near(0);
            if (n_units) start_units(b - 1);
            load_diag(b + 1);
            load_orig(j0 + QB);
        }
        // block b - 1's errors to memory
        if (b > 0) write_errors(b - 1);
        // the deferred products, then, as they come, the walked tiles' into the next block; those of the last are left for behind the walk
        units(b - 1, std::integral_constant<int, 0>{}, n_units);
        if (later > 0)
            while (taken < NT - 1) {
                const int now = walked_tiles();
                if (now > taken) take(min(now, NT - 1)); else __builtin_amdgcn_s_sleep(2);
            }
        lds_barrier();                                  // the walk is over
        behind = later > 1;
        if (later > 0) {
            take(NT);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) head[rt] = acc[0][rt] + sum[rt];
            if (later > 1 && group_starts(b + 1)) {     // the group's range wants all of its blocks as they stand
                start_units(b);
                units(b, std::integral_constant<int, 1>{}, later - 1);
                behind = false;
            }
#pragma unroll
            for (int j = 0; j + 1 < STRIP_BLOCKS - 1; ++j)
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) acc[j][rt] = acc[j + 1][rt];
            hand_over(b + 1);
            __builtin_amdgcn_s_waitcnt(0x0F70);         // vmcnt(0): the next block's matrix is in LDS (the next barrier publishes it)
        }
    }
    write_errors(nblocks - 1);
}

template <int FORM, int RT>
void launch_rows(const StripArgs& g, hipStream_t s) {
    hipLaunchKernelGGL((alg1_strip_kernel<FORM, RT>), dim3((unsigned)ceil_div(g.r, 16 * RT)), dim3(64 * STRIP_WAVES), 0, s, g);
}
template <int FORM>
void launch_form(int rt, const StripArgs& g, hipStream_t s) {
    if (rt == 1) launch_rows<FORM, 1>(g, s);
    else if (rt == 3) launch_rows<FORM, 3>(g, s);
    else launch_rows<FORM, 2>(g, s);                    // four row tiles per CU are two strips of two
}

}  // namespace

int launch_pack_factor(const float* M, int64_t ldm, const float* D, int64_t ldd, bool diag_dense, int64_t n, int64_t j_first, bool with_pairs,
                       float* packed, hipStream_t s) {
    const int64_t j_last = std::min<int64_t>(n, j_first + STRIP_PACK_OUTER * STRIP_BLOCKS * QB);
    const int64_t nblk = ceil_div(j_last - j_first, QB), tiles = with_pairs ? 2 * PAIRS * ceil_div(nblk, STRIP_BLOCKS) : 0;
    hipLaunchKernelGGL(pack_factor_kernel, dim3((unsigned)(nblk * DIAG_PARTS + tiles)), dim3(256), 0, s, M, ldm, D, ldd, (int)diag_dense, n, j_first, (int)nblk, packed,
                       packed + STRIP_PACK_DIAG_BYTES / sizeof(float));
    GPTQ_LAUNCH_CHECK();
    return GPTQ_OK;
}

int launch_alg1_strip(bool rf, bool hybrid, const StripArgs& g, hipStream_t s) {
    const int rt = strip_row_tiles(hybrid ? FORM_HYBRID : (rf ? FORM_R : FORM_U), g.r);
    if (hybrid) launch_form<FORM_HYBRID>(rt, g, s);
    else if (rf) launch_form<FORM_R>(rt, g, s);
    else launch_form<FORM_U>(rt, g, s);
    GPTQ_LAUNCH_CHECK();
    return GPTQ_OK;
}

}  // namespace gptq
