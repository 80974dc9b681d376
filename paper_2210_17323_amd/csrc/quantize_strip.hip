// Step 3, the columns of one outer block (Algorithm 1, Section 3 Steps 1-3): a workgroup takes a strip of weight rows
// through all the blocks of 128 columns of an outer block of up to 1024 columns in ONE launch.  Rows are independent in
// Alg. 1 (the Hessian information is shared by all rows), so nothing crosses workgroups.
//
//   * The strip's working values -- RT * 16 rows x 1024 columns -- live in registers, as the accumulators of
//     v_mfma_f32_16x16x4_f32: of every block of 128 columns wavefront w owns columns 32 w .. 32 w + 31.  The update of the
//     later blocks, acc[later] += E_b M[b, later], reads E_b from LDS (A operand) and M straight from memory (B operand:
//     a workgroup uses every element of M once, so LDS would add nothing); acc[i] of one block becomes acc[i - 1] of
//     the next, where its products are summed.
//   * A block is walked by one wavefront per 16 rows: the 16 lanes of a DPP row are 16 weight rows, the four DPP rows
//     share the columns of those 16 rows, DPP row c holding columns 4 i + c in register i.  Four columns at a time
//     (a "quad", register i of the four DPP rows) are broadcast to all lanes and walked there redundantly -- grid value,
//     error, update of the quad's later columns --, then every lane updates its own later columns with the quad's four
//     errors.  Row j of the block's triangular matrix is read from LDS 64 values at a time, one ds_read_b32 for 16
//     registers of all four DPP rows: lane l of DPP row c receives M[j][4 (16 t + l) + c], and the multiply-add of
//     register 16 t + l picks it up with the DPP row broadcast.
//
// What bounds it: a column is ~17 instructions that depend on one another in a chain plus 16 multiply-adds on average, all
// of one wavefront (~210 cycles); a block's update is RT * 64 matrix instructions per later block and wavefront.  An
// outer block takes 144 / 181 / 232 / 308 us with 16 / 32 / 48 / 64 rows per workgroup (driven by R; strip_row_tiles has all forms),
// 100 of them in the walk.  With one lane per row, a launch per block and an update launch between blocks the walk was 86
// instructions per column for a quarter of the wavefronts, and an outer block of 4096 rows took ~600 us; Alg. 1 on a 4096 x 4096
// layer 2.88 -> 1.08 ms, 12288 x 12288 16.8 -> 13.3 ms, 14336 x 14336 in groups of 128 24.1 -> 21.3 ms, 3000 x 5120 in groups of 1024
// 3.92 -> 1.48 ms.
#include "quantize_common.h"

#include <utility>

namespace gptq {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

namespace {

constexpr int NQ = QB / 4;              // quads of columns in a block: registers per lane
constexpr int PW = QB + 4;              // pitch of the row buffers: 16 rows start on 16 different bank quads
constexpr int STRIP_BLOCKS = 8;         // blocks of an outer block
constexpr int PAIRS = STRIP_BLOCKS * (STRIP_BLOCKS - 1) / 2;
// A block's triangular matrix, as it lies in LDS and (packed once per call) in the workspace: rows 0..63 whole, of rows
// 64..127 only columns 64..127, then for every quad of columns the values the quad's own walk needs, 16 floats:
// M01 M02 M03 M12, M13 M23 - -, the diagonal M00 M11 M22 M33, and the hardware's reciprocal estimates of the diagonal.
constexpr int DIAG_FAR = 64 * QB + 64 * 64;
constexpr int DIAG_WORDS = DIAG_FAR + NQ * 16;
constexpr int diag_row(int j) { return j < 64 ? j * QB : 64 * QB + (j - 64) * 64 - 64; }
constexpr int PAIR_WORDS = QB * QB;
static_assert(STRIP_DIAG_BYTES == DIAG_WORDS * 4 && STRIP_PAIR_BYTES == (size_t)PAIRS * PAIR_WORDS * 4, "quantize_common.h states these sizes");

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
    float w[NQ];                        // columns 4 i + c of this lane's row
    floatx4 n0[2], nd[2], nr[2];        // M01 M02 M03 M12, the diagonal and its reciprocals (this quad, next quad)
    floatx2 n1[2];                      // M13 M23
    floatx4 orig[2];                    // original weights of the quad's columns (R and hybrid forms)
    float ring[2][8];                   // row 4 i + a, half t: element [2 a + t], spread over the lanes
    RowGrid grid;
    float maxq, e2;
    lds_float lane_diag;                // block matrix + this lane's element of every half row
    lds_float diag;
    lds_float orow;                     // this row of the original weights
    lds_float erow;                     // this row of the strip's error block
    uint32_t __attribute__((address_space(3)))* crow;      // this row's codes, four to a word
    bool writer;                        // DPP row 0
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
        for (int a = 0; a < 4; ++a) {
            if constexpr (I < 15) s.ring[I & 1][2 * a] = *(lds_float_ordered)(s.lane_diag + diag_row(4 * I + a));
            if constexpr (I < 31) s.ring[I & 1][2 * a + 1] = *(lds_float_ordered)(s.lane_diag + diag_row(4 * I + a) + 64);
        }
    }
}

// w += ne * (element C of u's DPP row), for all lanes.  The s_nop covers the wait states a DPP read needs after a
// vector write of the same register, should the compiler have moved the row there.
template <int C, bool FIRST>
__device__ __forceinline__ void fma_row_bcast(float& w, float u, float ne) {
    if constexpr (FIRST)
        asm volatile("s_nop 1\n\tv_fmac_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(w) : "v"(u), "v"(ne), "n"(C));
    else
        asm volatile("v_fmac_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(w) : "v"(u), "v"(ne), "n"(C));
}

template <int FIRST_REG, int T, int FORM, int... C>
__device__ __forceinline__ void far_half(Walk<FORM>& s, float u, float ne, std::integer_sequence<int, C...>) {
    constexpr int first = FIRST_REG > 16 * T ? FIRST_REG - 16 * T : 0;
    ((C >= first ? fma_row_bcast<C, C == first>(s.w[16 * T + C], u, ne) : (void)0), ...);
}

// the lane's value of DPP rows 0 .. 3, in every DPP row
__device__ __forceinline__ void bcast_rows(float v, float (&x)[4]) {
    asm volatile("s_nop 3" : "+v"(v));          // v was last written by a statement the compiler cannot see into
    const uint32_t u = __float_as_uint(v);
    const auto h = __builtin_amdgcn_permlane32_swap(u, u, false, false);         // {rows 0 1 0 1, rows 2 3 2 3}
    const auto lo = __builtin_amdgcn_permlane16_swap(h[0], h[0], false, false);  // {rows 0 0 0 0, rows 1 1 1 1}
    const auto hi = __builtin_amdgcn_permlane16_swap(h[1], h[1], false, false);
    x[0] = __uint_as_float(lo[0]); x[1] = __uint_as_float(lo[1]);
    x[2] = __uint_as_float(hi[0]); x[3] = __uint_as_float(hi[1]);
}

// Grid of the group of 4 * LEN columns that starts at quad I, from the weights as they stand
template <int I, int LEN, int FORM>
__device__ __forceinline__ void group_grid(Walk<FORM>& s, int grid) {
    float lo = s.w[I], hi = s.w[I];
#pragma unroll
    for (int k = 1; k < LEN; ++k) { lo = fminf(lo, s.w[I + k]); hi = fmaxf(hi, s.w[I + k]); }
    float l4[4], h4[4];
    bcast_rows(lo, l4);
    bcast_rows(hi, h4);
    lo = fminf(fminf(l4[0], l4[1]), fminf(l4[2], l4[3]));
    hi = fmaxf(fmaxf(h4[0], h4[1]), fmaxf(h4[2], h4[3]));
    float sc; int zr;
    grid_from_range(grid, s.maxq, lo, hi, fmaxf(fabsf(lo), fabsf(hi)), sc, zr);
    s.grid.set(sc, zr, s.maxq);
}

struct GroupOut { float* scales; int32_t* zeros; };        // this row's first group of the block

template <int I, int FORM>
__device__ __forceinline__ void walk_quad(Walk<FORM>& s, int in_group, int kind, int nbk, const GroupOut& go) {
    request_quad<I + 1, FORM>(s);
    if constexpr (FORM != FORM_R) {
        // a group starts here (in_group: columns of a group inside the block, 0 otherwise; the same for all lanes)
        bool start = false;
        if constexpr (I % 2 == 0) { if (in_group == 8) { group_grid<I, 2>(s, kind); start = true; } }
        if constexpr (I % 4 == 0) { if (in_group == 16) { group_grid<I, 4>(s, kind); start = true; } }
        if constexpr (I % 8 == 0) { if (in_group == 32) { group_grid<I, 8>(s, kind); start = true; } }
        if constexpr (I % 16 == 0) { if (in_group == 64) { group_grid<I, 16>(s, kind); start = true; } }
        if constexpr (I == 0) { if (in_group == 128) { group_grid<I, 32>(s, kind); start = true; } }
        if constexpr (I % 2 == 0) {
            if (start && 4 * I < nbk && s.writer && go.scales) {
                const int gi = (4 * I) / in_group;
                go.scales[gi] = s.grid.scale;
                go.zeros[gi] = s.grid.zero;
            }
        }
    }
    float x[4];
    bcast_rows(s.w[I], x);
    floatx4 out;
    float t[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        const float mjj = s.nd[I & 1][a], rcp = s.nr[I & 1][a];
        float e, ne;
        if constexpr (FORM == FORM_R) {
            // the weight Alg. 1 holds here is w_j + s_j / R_jj: reciprocal estimate and one correction step with the exact
            // remainder (R_jj is the square root of a pivot of the damped Hessian: no range scaling needed)
            const float t0 = x[a] * rcp;
            const float wj = s.orig[I & 1][a];
            const float wn = wj + fmaf(fmaf(-t0, mjj, x[a]), rcp, t0);
            t[a] = s.grid.decide(wn);
            const float cz = t[a] - MAGIC;                                  // code - zero; the grid value is scale * cz
            ne = fmaf(-s.grid.scale, cz, wj);                               // d_j
            e = fmaf(-s.grid.scale, cz, wn) * mjj;
            out[a] = ne;
        } else {
            t[a] = s.grid.decide(x[a]);
            const float cz = t[a] - MAGIC;
            // e = (w - q) / U_jj in the same way
            const float d = fmaf(s.grid.scale, cz, -x[a]);                  // q - w
            const float e0 = d * rcp;
            e = ne = fmaf(fmaf(-e0, mjj, d), rcp, e0);                      // -e: only its square is wanted besides
            out[a] = FORM == FORM_U ? ne : fmaf(-s.grid.scale, cz, s.orig[I & 1][a]);
        }
        s.e2 = fmaf(e, e, s.e2);
        asm volatile("" : "+v"(s.e2));          // made here: sunk to the end of the walk, its operands would stay in registers
        if (a == 0) { x[1] = fmaf(ne, s.n0[I & 1][0], x[1]); x[2] = fmaf(ne, s.n0[I & 1][1], x[2]); x[3] = fmaf(ne, s.n0[I & 1][2], x[3]); }
        if (a == 1) { x[2] = fmaf(ne, s.n0[I & 1][3], x[2]); x[3] = fmaf(ne, s.n1[I & 1][0], x[3]); }
        if (a == 2) x[3] = fmaf(ne, s.n1[I & 1][1], x[3]);
        if constexpr (I < 15) far_half<I + 1, 0>(s, s.ring[I & 1][2 * a], ne, std::make_integer_sequence<int, 16>{});
        if constexpr (I < 31) far_half<I + 1, 1>(s, s.ring[I & 1][2 * a + 1], ne, std::make_integer_sequence<int, 16>{});
    }
    // the four low bytes, side by side
    const uint32_t c01 = __builtin_amdgcn_perm(__float_as_uint(t[1]), __float_as_uint(t[0]), 0x0c0c0400u);
    const uint32_t c23 = __builtin_amdgcn_perm(__float_as_uint(t[3]), __float_as_uint(t[2]), 0x04000c0cu);
    const uint32_t code = (c01 | c23) - s.grid.bias;
    if (s.writer) {
        *(__attribute__((address_space(3))) floatx4*)(s.erow + 4 * I) = out;
        s.crow[I] = code;
    }
}

template <int FORM, int... I>
__device__ __forceinline__ void walk_block(Walk<FORM>& s, int in_group, int kind, int nbk, const GroupOut& go, std::integer_sequence<int, I...>) {
    request_quad<0, FORM>(s);
    (walk_quad<I, FORM>(s, in_group, kind, nbk, go), ...);
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

// STRIP_PACK_OUTER outer blocks of the factor, from column j_first on, as the strip kernel reads them.  Workgroups 0 ..
// nblk - 1: one diagonal block each (identity outside the matrix).  Then two per 128 x 128 tile above the diagonal blocks of an outer block (64 rows each), in the
// order in which the lanes take B operands: [wavefront: 32 columns][16 rows][even, odd columns][lane][4 rows], zeros outside
// the matrix.  Read as it lies, 128 columns of a factor whose rows are a multiple of 4 KB apart come from two of an
// XCD's sixteen L2 channels, with every CU of the chip reading the same 512 bytes of each row at the same time.
__global__ __launch_bounds__(256) void pack_factor_kernel(const float* M, int64_t ldm, const float* D, int64_t ldd, int diag_dense,
                                                          int64_t n, int64_t j_first, int nblk, float* diag_out, float* pair_out) {
    __shared__ float tile[64][QB + 1];
    const int tid = threadIdx.x;
    if ((int)blockIdx.x < nblk) {
        const int64_t j0 = j_first + (int64_t)blockIdx.x * QB;
        const float* B = D + (diag_dense ? j0 * QB : j0 * ldd + j0);
        const int64_t ld = diag_dense ? QB : ldd;
        const int lim = diag_dense ? QB : (int)min((int64_t)QB, n - j0);
        float* out = diag_out + (int64_t)blockIdx.x * DIAG_WORDS;
        auto at = [&](int j, int k) { return (j < lim && k < lim) ? B[j * ld + k] : (j == k ? 1.f : 0.f); };
        for (int q = tid; q < DIAG_FAR; q += 256) {
            const int j = q < 64 * QB ? q >> 7 : 64 + ((q - 64 * QB) >> 6), k = q < 64 * QB ? q & 127 : 64 + ((q - 64 * QB) & 63);
            out[q] = at(j, k);
        }
        for (int q = tid; q < NQ * 16; q += 256) {
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
    const int p = ((int)blockIdx.x - nblk) >> 1, h = ((int)blockIdx.x - nblk) & 1;
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
    for (int i = tid; i < 64 * 32; i += 256) {              // 16-byte pieces of this half: [wavefront][4 row groups][2][lane]
        const int lane = i & 63, ct = (i >> 6) & 1, t = (i >> 7) & 3, w = i >> 9;
        const int col = 32 * w + 2 * (lane & 15) + ct, k = 16 * t + 4 * (lane >> 4);
        const floatx4 v = {tile[k][col], tile[k + 1][col], tile[k + 2][col], tile[k + 3][col]};
        *reinterpret_cast<floatx4*>(out + (((w * 8 + 4 * h + t) * 2 + ct) * 64 + lane) * 4) = v;
    }
}

// A barrier that orders LDS accesses only: __syncthreads() would also wait for every global access in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int FORM, int RT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void alg1_strip_kernel(StripArgs g) {
    constexpr int ROWS = 16 * RT;
    __shared__ __attribute__((aligned(16))) float diag[DIAG_WORDS];
    __shared__ __attribute__((aligned(16))) float ebuf[ROWS * PW];         // the block's working values, then its errors
    __shared__ __attribute__((aligned(16))) float obuf[FORM == FORM_U ? 4 : ROWS * PW];     // the block's original weights
    __shared__ __attribute__((aligned(16))) uint32_t cbuf[ROWS * NQ];      // codes
    __shared__ float red[2][4][FORM == FORM_U ? ROWS : 1];                 // group ranges of the four wavefronts

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, kq = lane >> 4;
    const int64_t row0 = (int64_t)blockIdx.x * ROWS;
    const int nblocks = (int)((g.o1 - g.o0 + QB - 1) / QB);

    // ---- the strip's working values of all blocks: lane (l16, kq) of wavefront w holds columns 32 w + 2 l16 + {0, 1} of
    //      rows 16 rt + 4 kq + e.  Rows past r repeat the last one and are never stored; columns past the outer block are zero.
    floatx4 acc[STRIP_BLOCKS][RT][2];
    const int wcol = 32 * wave + 2 * l16;
    {
        // addresses: a base that is the same for all lanes and 32-bit offsets (64 rows of the working matrix are below 4 GiB)
        uint32_t off[RT][4];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int rr = (int)min((int64_t)(16 * rt + 4 * kq + e), g.r - 1 - row0);
                off[rt][e] = ((uint32_t)rr * (uint32_t)g.lds_ + (uint32_t)wcol) * 4u;
            }
        const char* base = reinterpret_cast<const char*>(g.S + row0 * g.lds_ + g.o0);
#pragma unroll
        for (int i = 0; i < STRIP_BLOCKS; ++i) {
            const int64_t left = strip_block_columns(g.o0, g.o1, i);
            if (!g.S || left <= 0) {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) acc[i][rt][0] = acc[i][rt][1] = floatx4{0.f, 0.f, 0.f, 0.f};
            } else if (left >= QB) {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const floatx2 v = *reinterpret_cast<const floatx2*>(base + i * (QB * 4) + off[rt][e]);
                        acc[i][rt][0][e] = v[0];
                        acc[i][rt][1][e] = v[1];
                    }
            } else {
                const bool in0 = wcol < left, in1 = wcol + 1 < left;
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const char* p = base + i * (QB * 4) + off[rt][e];
                        const float v0 = *reinterpret_cast<const float*>(in0 ? p : base), v1 = *reinterpret_cast<const float*>(in1 ? p + 4 : base);
                        acc[i][rt][0][e] = in0 ? v0 : 0.f;
                        acc[i][rt][1][e] = in1 ? v1 : 0.f;
                    }
            }
        }
    }

    // ---- staging of a block: its triangular matrix (identity outside the matrix) and its original weights
    auto load_diag = [&](int64_t j0) {
        // straight into LDS, 1 KB per wavefront and instruction
        const float* src = g.diag + (j0 - g.o0) / QB * DIAG_WORDS + tid * 4;
#pragma unroll
        for (int t = 0; t < DIAG_WORDS / 1024; ++t)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + 1024 * t),
                                             (__attribute__((address_space(3))) void*)(diag + 1024 * t + 256 * wave), 16, 0, 0);
        if (wave < (DIAG_WORDS % 1024) / 256)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + DIAG_WORDS / 1024 * 1024),
                                             (__attribute__((address_space(3))) void*)(diag + DIAG_WORDS / 1024 * 1024 + 256 * wave), 16, 0, 0);
    };
    // The original weights are requested as they are and turned into float32 only when they are put into LDS, so that
    // nothing waits for them in between.  Rows that cannot be read four weights at a time are read there, one by one.
    floatx4 oreg[FORM == FORM_U ? 1 : 2 * RT];
    auto orig_whole = [&](int64_t j0) { return g.w_vec && j0 + QB <= g.n; };
    auto orig_at = [&](int64_t j0, int t) {
        const int q = tid + 256 * t;
        return min(row0 + (q >> 5), g.r - 1) * g.ldw + j0 + (q & 31) * 4;
    };
    auto load_orig = [&](int64_t j0) {
        if constexpr (FORM != FORM_U) {
            if (!orig_whole(j0)) return;
            if (g.wdtype == GPTQ_F32) {
#pragma unroll
                for (int t = 0; t < 2 * RT; ++t) oreg[t] = *reinterpret_cast<const floatx4*>(static_cast<const float*>(g.W) + orig_at(j0, t));
            } else {
#pragma unroll
                for (int t = 0; t < 2 * RT; ++t) {
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
            for (int t = 0; t < 2 * RT; ++t) {
                const int q = tid + 256 * t, k = (q & 31) * 4;
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
    load_diag(g.o0);
    load_orig(g.o0);
    store_orig(g.o0);

    const int64_t wrow = row0 + 16 * wave + l16;                     // the row this lane walks (wavefronts 0 .. RT - 1)
    const int64_t wrow_c = min(wrow, g.r - 1);
    Walk<FORM> s;
    s.maxq = (float)g.maxq;
    s.grid.set(1.f, 0, s.maxq);
    double half = 0.0;
    if (wave < RT) {
        if (g.in_group == 0 && g.wide_group == 0) {
            const int64_t gi = wrow_c * g.ngroups + (g.group ? g.o0 / g.group : 0);
            s.grid.set(g.scales[gi], g.zeros[gi], s.maxq);
        }
        if (g.half_e2 && g.o0 > 0) half = g.half_e2[wrow_c];
        s.writer = kq == 0;
        s.diag = (lds_float)diag;
        s.lane_diag = s.diag + 4 * l16 + kq;
        s.erow = (lds_float)ebuf + (16 * wave + l16) * PW;
        s.orow = FORM == FORM_U ? s.erow : (lds_float)obuf + (16 * wave + l16) * PW;
        s.crow = (uint32_t __attribute__((address_space(3)))*)cbuf + (16 * wave + l16) * NQ;
    }

#pragma unroll 1
    for (int b = 0; b < nblocks; ++b) {
        const int64_t j0 = g.o0 + (int64_t)b * QB;
        const int nbk = (int)min((int64_t)QB, g.n - j0);
        // ---- the block's working values to the walkers
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const floatx2 v = {acc[0][rt][0][e], acc[0][rt][1][e]};
                *reinterpret_cast<floatx2*>(&ebuf[(16 * rt + 4 * kq + e) * PW + wcol]) = v;
            }
        if constexpr (FORM == FORM_U) {
            // a group of several blocks starts here: its range over the current values of all its columns
            if (g.wide_group && (j0 % g.wide_group) == 0) {
                const int gb = (int)(g.wide_group / QB);
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        float lo = acc[0][rt][0][e], hi = lo;
#pragma unroll
                        for (int i = 0; i < STRIP_BLOCKS; ++i)
                            if (i < gb) {
                                lo = fminf(lo, fminf(acc[i][rt][0][e], acc[i][rt][1][e]));
                                hi = fmaxf(hi, fmaxf(acc[i][rt][0][e], acc[i][rt][1][e]));
                            }
#pragma unroll
                        for (int o = 8; o > 0; o >>= 1) { lo = fminf(lo, __shfl_xor(lo, o)); hi = fmaxf(hi, __shfl_xor(hi, o)); }
                        if (l16 == 0) { red[0][wave][16 * rt + 4 * kq + e] = lo; red[1][wave][16 * rt + 4 * kq + e] = hi; }
                    }
            }
        }
        if (b == 0) __builtin_amdgcn_s_waitcnt(0x0F70);             // vmcnt(0): the first block's copies into LDS have landed
        lds_barrier();
        // ---- the walk
        if (wave < RT) {
            if constexpr (FORM == FORM_U) {
                if (g.wide_group && (j0 % g.wide_group) == 0) {
                    const int rr = 16 * wave + l16;
                    const float lo = fminf(fminf(red[0][0][rr], red[0][1][rr]), fminf(red[0][2][rr], red[0][3][rr]));
                    const float hi = fmaxf(fmaxf(red[1][0][rr], red[1][1][rr]), fmaxf(red[1][2][rr], red[1][3][rr]));
                    float sc; int zr;
                    grid_from_range(g.grid, s.maxq, lo, hi, fmaxf(fabsf(lo), fabsf(hi)), sc, zr);
                    s.grid.set(sc, zr, s.maxq);
                    if (s.writer && wrow < g.r) {
                        g.scales[wrow * g.ngroups + j0 / g.wide_group] = sc;
                        g.zeros[wrow * g.ngroups + j0 / g.wide_group] = zr;
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < NQ; ++i) {
                s.w[i] = s.erow[4 * i + kq];
                if constexpr (FORM == FORM_HYBRID) s.w[i] += s.orow[4 * i + kq];
            }
            s.e2 = 0.f;
            GroupOut go{nullptr, nullptr};
            if (g.in_group && wrow < g.r) {
                const int64_t gi = wrow * g.ngroups + j0 / g.in_group;
                go.scales = g.scales + gi;
                go.zeros = g.zeros + gi;
            }
            walk_block<FORM>(s, g.in_group, g.grid, nbk, go, std::make_integer_sequence<int, NQ>{});
            half += 0.5 * (double)s.e2;
        }
        lds_barrier();
        // ---- the later blocks, and what leaves: errors and codes
        const int later = nblocks - 1 - b;
        if (later > 0) {
            // B fragments: step (t, e) pairs element k = 16 t + 4 kq + e of E with row k of M; half a block (four t) is in
            // flight while the other half is multiplied.  Past the last half the loads repeat it.
            const int first_pair = b * (2 * STRIP_BLOCKS - 1 - b) / 2;           // pair (b, b + 1) of the packed tiles
            const float* tiles = g.pairs + first_pair * PAIR_WORDS + wave * (8 * 2 * 256) + lane * 4;
            constexpr int AHEAD = RT == 1 ? 3 : 2;                   // buffers of B halves: AHEAD - 1 halves in flight beside the one in use
            floatx4 bf[AHEAD][4][2];
            auto request = [&](int h, floatx4 (&dst)[4][2]) {
                const int hc = min(h, 2 * later - 1);
                const float* p = tiles + (hc >> 1) * PAIR_WORDS + (hc & 1) * (4 * 2 * 256);
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int ct = 0; ct < 2; ++ct) dst[t][ct] = *reinterpret_cast<const floatx4*>(p + (t * 2 + ct) * 256);
            };
            // A fragments: the same for all later blocks, so a small strip reads them once; a large one, short of registers,
            // reads them again for every block beside its longer run of products.
            constexpr bool A_ONCE = RT <= 2;
            const float* arow = &ebuf[l16 * PW + 4 * kq];
            floatx4 af[A_ONCE ? 8 : 1][RT];
            if constexpr (A_ONCE) {
#pragma unroll
                for (int t = 0; t < 8; ++t)
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt) af[t][rt] = *reinterpret_cast<const floatx4*>(arow + 16 * rt * PW + 16 * t);
            }
            auto multiply = [&](int half_, const floatx4 (&src)[4][2], floatx4 (&d)[RT][2]) {
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    floatx4 a[RT];
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt) {
                        if constexpr (A_ONCE) a[rt] = af[4 * half_ + t][rt];
                        else a[rt] = *reinterpret_cast<const floatx4*>(arow + 16 * rt * PW + 64 * half_ + 16 * t);
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                            for (int ct = 0; ct < 2; ++ct)
                                d[rt][ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[rt][e], src[t][ct][e], (half_ == 0 && t == 0 && e == 0) ? floatx4{0.f, 0.f, 0.f, 0.f} : d[rt][ct], 0, 0, 0);
                }
            };
            // The fences keep every request ahead of the products it runs beside (left alone, the compiler moves the loads
            // down to their uses and waits for each).
#pragma unroll
            for (int h = 0; h < AHEAD - 1; ++h) request(h, bf[h]);
            __builtin_amdgcn_sched_barrier(0);
            load_diag(j0 + QB);                 // the walkers left the block's matrix and weights at the barrier above
            load_orig(j0 + QB);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 1; i < STRIP_BLOCKS; ++i) {
                if (i <= later) {
                    const int h = 2 * (i - 1);
                    request(h + AHEAD - 1, bf[(h + AHEAD - 1) % AHEAD]);
                    __builtin_amdgcn_sched_barrier(0);
                    multiply(0, bf[h % AHEAD], acc[i - 1]);
                    __builtin_amdgcn_sched_barrier(0);
                    request(h + AHEAD, bf[h % AHEAD]);
                    __builtin_amdgcn_sched_barrier(0);
                    multiply(1, bf[(h + 1) % AHEAD], acc[i - 1]);
                    // The block's 128 products are summed on their own, in the place the block moves to, and added once.  Taken one by
                    // one, each is rounded at the size of the running value: the error sums E driven by U were 3.4 times as far
                    // from 64 bits, for 1 % (four row tiles, which then spill: 2 to 7 %) of the time.
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt) { acc[i - 1][rt][0] += acc[i][rt][0]; acc[i - 1][rt][1] += acc[i][rt][1]; }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            store_orig(j0 + QB);
            __builtin_amdgcn_s_waitcnt(0x0F70);             // vmcnt(0): the next block's matrix is in LDS (the barrier below publishes it)
        }
#pragma unroll
        for (int t = 0; t < 2 * RT; ++t) {
            const int q = tid + 256 * t, rr = q >> 5, k = (q & 31) * 4;
            if (row0 + rr < g.r && g.E) *reinterpret_cast<floatx4*>(g.E + (row0 + rr) * g.lde + (j0 - g.o0) + k) = *reinterpret_cast<const floatx4*>(&ebuf[rr * PW + k]);
        }
        for (int q = tid; q < ROWS * 8; q += 256) {
            const int rr = q >> 3, k = (q & 7) * 16;
            if (row0 + rr >= g.r) continue;
            uint8_t* dst = g.codes + (row0 + rr) * g.ldc + j0 + k;
            const uint4 v = *reinterpret_cast<const uint4*>(&cbuf[rr * NQ + (k >> 2)]);
            if (k + 16 <= nbk && (reinterpret_cast<uintptr_t>(dst) & 15) == 0) {
                *reinterpret_cast<uint4*>(dst) = v;
            } else {
                const uint32_t wds[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int c = 0; c < 16; ++c)
                    if (k + c < nbk) dst[c] = (uint8_t)(wds[c >> 2] >> (8 * (c & 3)));
            }
        }
        lds_barrier();                  // everybody has read the errors and codes of this block
    }
    if (wave < RT && kq == 0 && wrow < g.r && g.half_e2) g.half_e2[wrow] = half;
}

template <int FORM>
void launch_form(int rt, const StripArgs& g, hipStream_t s) {
    const dim3 grid((unsigned)ceil_div(g.r, 16 * rt));
    switch (rt) {
        case 1:  hipLaunchKernelGGL((alg1_strip_kernel<FORM, 1>), grid, dim3(256), 0, s, g); break;
        case 2:  hipLaunchKernelGGL((alg1_strip_kernel<FORM, 2>), grid, dim3(256), 0, s, g); break;
        case 3:  hipLaunchKernelGGL((alg1_strip_kernel<FORM, 3>), grid, dim3(256), 0, s, g); break;
        default: hipLaunchKernelGGL((alg1_strip_kernel<FORM, 4>), grid, dim3(256), 0, s, g); break;
    }
}

}  // namespace

int launch_pack_factor(const float* M, int64_t ldm, const float* D, int64_t ldd, bool diag_dense, int64_t n, int64_t j_first, bool with_pairs,
                       float* packed, hipStream_t s) {
    const int64_t j_last = std::min<int64_t>(n, j_first + STRIP_PACK_OUTER * STRIP_BLOCKS * QB);
    const int64_t nblk = ceil_div(j_last - j_first, QB), tiles = with_pairs ? 2 * PAIRS * ceil_div(nblk, STRIP_BLOCKS) : 0;
    hipLaunchKernelGGL(pack_factor_kernel, dim3((unsigned)(nblk + tiles)), dim3(256), 0, s, M, ldm, D, ldd, (int)diag_dense, n, j_first, (int)nblk, packed,
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
