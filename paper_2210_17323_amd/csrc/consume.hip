// Consumers of the packed format (Section 4, "Practical Speedups", and the appendix on the benchmarking
// setup): the full-matrix decompression used before a large-batch product, and the quantized-matrix times
// full-precision-vector product of batch-1 generation, which dequantizes weights as it reads them and does
// not quantize the vector.  Both are bound by HBM: the packed words are read once.
//
// Layout (same as pack.hip): per row, code k occupies bits [k*b, (k+1)*b) of a little-endian stream of uint32
// words; 32 codes are exactly b words.  A weight is scale * (code - zero) with the scale and zero point of its
// row (group == 0) or of its row's group k / group.
#include "common.h"

#include <hip/hip_fp16.h>

#include <atomic>

namespace gptq {

struct PackedArgs {
    const uint32_t* words; int64_t ldp;
    int64_t r, n, words_per_row;
    const float* scales; const int32_t* zeros;
    int64_t group, ngroups;      // group == 0: one grid per row (ngroups == 1)
    int gshift;                  // log2(group) if the group size is a power of two, else -1 (then columns are divided)
    int64_t rows_per_wg;         // matvec: rows a workgroup walks, a multiple of its row chunk
    int segw, segshift;          // matvec: wavefronts that share a row, each every segw-th segment of columns; segw = 1 << segshift
};

template <int BITS>
__device__ __forceinline__ uint32_t code_at(const uint32_t (&w)[BITS], int i) {
    const int pos = i * BITS, wi = pos >> 5, off = pos & 31;
    uint32_t v = w[wi] >> off;
    if (off + BITS > 32) v |= w[(wi + 1) % BITS] << (32 - off);      // % only keeps the index in range for the compiler
    return v & ((1u << BITS) - 1u);
}

// ---- codes to halves without a conversion (used by both consumers) -------------------------------------------------
// With the exponent bits of 2^b or-ed in, a code sitting at mantissa bits [10-b, 10) of a half IS the float16 number
// 2^b + code.  Two codes whose bit positions differ by 16 (mod 32) sit at the same place of the two halves of a
// 32-bit word, so one shift puts both at [10-b, 10) / [26-b, 26) and one and-or masks them and sets both exponents:
//   b = 4: codes k and k+4 of a word;  b = 2: codes k and k+8 of a word;
//   b = 3: codes k and k+16 of the 96-bit group are 48 bits apart -- low half of one word, high half of another,
//          joined by one byte permute that serves four or five pairs; the two pairs whose codes straddle a
//          16-bit boundary (5, 21 and 10, 26) are cut out one code at a time.
typedef _Float16 half2v __attribute__((ext_vector_type(2)));

struct PairSpec { int lo_word, hi_word, rel, k_lo, k_hi; };      // lo_word < 0: cut the two codes out one at a time
template <int BITS> struct PairTable;
template <> struct PairTable<4> {
    static constexpr PairSpec at(int i) { return {i / 4, i / 4, 4 * (i % 4), 8 * (i / 4) + i % 4, 8 * (i / 4) + i % 4 + 4}; }
};
template <> struct PairTable<2> {
    static constexpr PairSpec at(int i) { return {i / 8, i / 8, 2 * (i % 8), 16 * (i / 8) + i % 8, 16 * (i / 8) + i % 8 + 8}; }
};
template <> struct PairTable<3> {
    static constexpr PairSpec at(int i) {
        if (i < 5) return {0, 1, 3 * i, i, i + 16};                                   // k = 0..4
        if (i < 9) return {2, 0, 3 * (i + 1) - 16, (i + 1) + 16, i + 1};              // k = 6..9
        if (i < 14) return {1, 2, 3 * (i + 2) - 32, i + 2, (i + 2) + 16};             // k = 11..15
        return i == 14 ? PairSpec{-1, -1, 0, 5, 21} : PairSpec{-1, -1, 0, 10, 26};
    }
};

__device__ __forceinline__ uint32_t and_or(uint32_t a, uint32_t mask, uint32_t c) {
    uint32_t v;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(v) : "v"(a), "s"(mask), "v"(c));   // written out: the compiler spends two on it
    return v;
}

// 32 bits of the stream of words w[0..BITS] (w[BITS] = 0) starting at bit `from` (may be negative: shifted in zeros)
template <int BITS>
__device__ __forceinline__ uint32_t stream_bits(const uint32_t (&w)[BITS + 1], int from) {
    if (from < 0) return w[0] << (-from);
    const int wi = from >> 5, sh = from & 31;
    return sh ? __builtin_amdgcn_alignbit(w[wi + 1], w[wi], sh) : w[wi];
}


// The 32 codes of b words as 16 registers of two halves (2^b + code each); register i holds codes PairTable::at(i).k_lo
// (low half) and .k_hi (high half).  w[BITS] must be 0.
template <int BITS>
__device__ __forceinline__ void codes_as_half_pairs(const uint32_t (&w)[BITS + 1], uint32_t (&pr)[16]) {
    constexpr int WANT = 10 - BITS;
    constexpr uint32_t M = (1u << BITS) - 1u;
    constexpr uint32_t MASK_LO = M << WANT, MASK_HI = M << (16 + WANT), MASK = MASK_LO | MASK_HI;
    const uint32_t magic = 0x3C003C00u + (uint32_t)BITS * 0x04000400u;       // (2^b, 2^b) as two halves
    uint32_t joined[3] = {0u, 0u, 0u};
    if constexpr (BITS == 3) {
        joined[0] = __builtin_amdgcn_perm(w[1], w[0], 0x07060100u);      // low half of w0, high half of w1
        joined[1] = __builtin_amdgcn_perm(w[0], w[2], 0x07060100u);      // low half of w2, high half of w0
        joined[2] = __builtin_amdgcn_perm(w[2], w[1], 0x07060100u);      // low half of w1, high half of w2
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const PairSpec sp = PairTable<BITS>::at(i);
        if (sp.lo_word < 0) {
            const uint32_t ta = stream_bits<BITS>(w, BITS * sp.k_lo - WANT);
            const uint32_t tb = stream_bits<BITS>(w, BITS * sp.k_hi - (16 + WANT));
            pr[i] = and_or(tb, MASK_HI, and_or(ta, MASK_LO, magic));
        } else {
            uint32_t m;
            if (sp.lo_word == sp.hi_word) m = w[sp.lo_word];
            else m = joined[sp.lo_word == 0 ? 0 : (sp.lo_word == 2 ? 1 : 2)];
            const uint32_t t = sp.rel >= WANT ? (m >> (sp.rel - WANT)) : (m << (WANT - sp.rel));
            pr[i] = and_or(t, MASK, magic);
        }
    }
}

// ---- full-matrix decompression, the usual case (n a multiple of 8, one grid per 8 columns, 16-byte aligned rows) ----
// A workgroup walks along a row (then along every gridDim.x-th row after it), one thread per 8 codes per step:
// neighbouring lanes write neighbouring 16 bytes, so a store instruction of a wavefront covers 1 KB without a gap and a
// workgroup streams a whole row; lanes re-read words their neighbours also read (served by the vector cache).
// The 8 codes are 8 b consecutive bits of at most two words.  Or-ed into 0x6400 a code IS the half 1024 + code, so a
// pair of codes costs a shift and two and-ors, one packed subtraction of 1024 + zero leaves the exact integers
// code - zero, and each output is the float32 product with the scale, rounded to the output type.
template <int BITS, typename OT>
__global__ __launch_bounds__(256) void dequantize8_kernel(PackedArgs a, OT* __restrict__ out, int64_t ldo, int64_t octets_per_row) {
    constexpr uint32_t M = (1u << BITS) - 1u;
    constexpr int UN = 1;                       // octets per thread per step (256 apart; more in flight measured slower)
    for (int64_t row = blockIdx.x; row < a.r; row += gridDim.x) {
        const uint32_t* __restrict__ wrow = a.words + row * a.ldp;
        OT* orow = out + row * ldo;
        const float* srow = a.scales + row * a.ngroups;
        const int32_t* zrow = a.zeros + row * a.ngroups;
        for (int64_t oc0 = threadIdx.x; oc0 < octets_per_row; oc0 += 256 * UN) {
            uint32_t lo[UN], hi[UN];
            float sc[UN], zf[UN];
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int64_t oc = oc0 + 256 * u;
                lo[u] = hi[u] = 0u; sc[u] = 0.f; zf[u] = 0.f;
                if (oc < octets_per_row) {
                    const int64_t bit0 = oc * 8 * BITS, wi = bit0 >> 5;
                    const int off = (int)(bit0 & 31);
                    lo[u] = wrow[wi];
                    if ((off + 8 * BITS > 32) && (wi + 1 < a.words_per_row)) hi[u] = wrow[wi + 1];
                    // column / group size without the 64-bit division (n < 2^31 columns are checked on the host)
                    const uint32_t col = (uint32_t)(oc * 8);
                    const uint32_t gcol = a.group == 0 ? 0u : (a.gshift >= 0 ? col >> a.gshift : col / (uint32_t)a.group);
                    sc[u] = srow[gcol];
                    zf[u] = (float)zrow[gcol];
                }
            }
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int64_t oc = oc0 + 256 * u;
                if (oc >= octets_per_row) break;
                const int off = (int)((oc * 8 * BITS) & 31);
                const uint32_t bits8 = __builtin_amdgcn_alignbit(hi[u], lo[u], off);       // code i at bits [i*b, (i+1)*b)
                const _Float16 zh = (_Float16)(1024.f + zf[u]);                              // exact
                half2v z2; z2.x = zh; z2.y = zh;
                _Float16 d[8];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t t = bits8 >> (2 * i * BITS);                              // codes 2i and 2i+1 at the bottom
                    const uint32_t pair = and_or(t << (16 - BITS), M << 16, and_or(t, M, 0x64006400u));
                    const half2v v = __builtin_bit_cast(half2v, pair) - z2;
                    d[2 * i] = v.x; d[2 * i + 1] = v.y;
                }
                OT* dst = orow + oc * 8;
                if constexpr (sizeof(OT) == 2) {
                    union { uint4 u4; _Float16 h[8]; } pk;
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        float prod = sc[u] * (float)d[i];       // the float32 product, rounded, and only then the half: the
                        asm volatile("" : "+v"(prod));          // two must not be fused into one mixed-precision instruction
                        pk.h[i] = (_Float16)prod;
                    }
                    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
                    u32x4 v4; v4.x = pk.u4.x; v4.y = pk.u4.y; v4.z = pk.u4.z; v4.w = pk.u4.w;
                    __builtin_nontemporal_store(v4, reinterpret_cast<u32x4*>(dst));     // written once, not read again here
                } else {
                    typedef float f32x4 __attribute__((ext_vector_type(4)));
                    f32x4 a4 = {sc[u] * (float)d[0], sc[u] * (float)d[1], sc[u] * (float)d[2], sc[u] * (float)d[3]};
                    f32x4 b4 = {sc[u] * (float)d[4], sc[u] * (float)d[5], sc[u] * (float)d[6], sc[u] * (float)d[7]};
                    __builtin_nontemporal_store(a4, reinterpret_cast<f32x4*>(dst));
                    __builtin_nontemporal_store(b4, reinterpret_cast<f32x4*>(dst) + 1);
                }
            }
        }
    }
}

// ---- full-matrix decompression, any shape: one thread per 8 codes = 8 consecutive outputs (one 16-byte store of halves) ---
// 8 codes are 8*b consecutive bits starting at a multiple of 8 bits: at most two words.  Neighbouring lanes
// write neighbouring 16 bytes, and re-read words their neighbours also read (served by the vector cache).
template <int BITS, typename OT>
__global__ __launch_bounds__(256) void dequantize_kernel(PackedArgs a, OT* out, int64_t ldo, int64_t octets_per_row) {
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (gid >= a.r * octets_per_row) return;
    const int64_t row = gid / octets_per_row, oc = gid % octets_per_row;
    const int64_t k0 = oc * 8;
    const int64_t bit0 = k0 * BITS, wi = bit0 >> 5;
    const int off = (int)(bit0 & 31);
    const uint32_t* p = a.words + row * a.ldp + wi;
    const uint64_t lo = p[0];
    const uint64_t hi = (off + 8 * BITS > 32 && wi + 1 < a.words_per_row) ? p[1] : 0u;
    const uint32_t bits8 = (uint32_t)(((hi << 32) | lo) >> off);        // the 8 codes, code i at bits [i*b, (i+1)*b)
    const bool one_grid = (a.group == 0) || (a.group % 8 == 0);
    const int64_t gbase = row * a.ngroups;
    float sc = 0.f, zf = 0.f;
    if (one_grid) {
        const int64_t gi = a.group ? k0 / a.group : 0;
        sc = a.scales[gbase + gi];
        zf = (float)a.zeros[gbase + gi];
    }
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if (!one_grid && k0 + i < a.n) {
            const int64_t gi = (k0 + i) / a.group;
            sc = a.scales[gbase + gi];
            zf = (float)a.zeros[gbase + gi];
        }
        v[i] = sc * ((float)((bits8 >> (i * BITS)) & ((1u << BITS) - 1u)) - zf);
    }
    OT* dst = out + row * ldo + k0;
    if ((k0 + 8 <= a.n) && (reinterpret_cast<uintptr_t>(dst) & 15) == 0) {
        if constexpr (sizeof(OT) == 2) {
            union { uint4 u; __half h[8]; } pk;
#pragma unroll
            for (int i = 0; i < 8; ++i) pk.h[i] = __float2half_rn(v[i]);
            *reinterpret_cast<uint4*>(dst) = pk.u;
        } else {
            reinterpret_cast<float4*>(dst)[0] = make_float4(v[0], v[1], v[2], v[3]);
            reinterpret_cast<float4*>(dst)[1] = make_float4(v[4], v[5], v[6], v[7]);
        }
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (k0 + i < a.n) {
                if constexpr (sizeof(OT) == 2) dst[i] = __float2half_rn(v[i]);
                else dst[i] = v[i];
            }
    }
}

// ---- y = Q x, batch 1 -----------------------------------------------------------------------------------------
// A wavefront takes 4 (or 8) rows and every segw-th 2048-column segment of them: a lane holds the 32 vector entries of
// its 32 columns in registers (read once per segment, shared by all the rows), reads b consecutive words per row -- a
// wavefront reads 64*b*4 contiguous bytes of a row -- and accumulates  scale * (sum code*x - zero * sum x)  in float32.
// The lane sums of four rows are reduced across the wavefront by lane swaps and row rotations, and across the segw wavefronts
// that share them through LDS.
constexpr int MV_ROWS = 4;
constexpr int MV_SEG = 64 * 32;
constexpr int MV_MAX_WAVES = 16;

template <int CTRL>
__device__ __forceinline__ float add_rotated(float v) {
    return v + __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), CTRL, 0xf, 0xf, false));
}
// Sums over the wavefront of four values at once: every lane of a group of 16 gets the sum of value wave_sum_index(lane).
__device__ __forceinline__ float wave_sum4(float a, float b, float c, float d) {
    auto swap32 = [](float x, float y) {
        const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
        return __uint_as_float(t[0]) + __uint_as_float(t[1]);
    };
    const float ab = swap32(a, b), cd = swap32(c, d);        // lanes 0 .. 31: a (c), 32 .. 63: b (d), two lanes summed
    const auto t = __builtin_amdgcn_permlane16_swap(__float_as_uint(ab), __float_as_uint(cd), false, false);
    float v = __uint_as_float(t[0]) + __uint_as_float(t[1]); // groups of 16 lanes: a, c, b, d
    v = add_rotated<0x128>(v);                               // row_ror 8, 4, 2, 1
    v = add_rotated<0x124>(v);
    v = add_rotated<0x122>(v);
    return add_rotated<0x121>(v);
}
__device__ __forceinline__ int wave_sum_index(int lane) { return ((lane >> 4) & 1) * 2 + (lane >> 5); }

// sum over the segw wavefronts of a row group, two at a time
template <int W>
__device__ __forceinline__ float sum_parts(const float (*part)[W], int first, int segw, int i) {
    float v = segw == 1 ? part[first][i] : part[first][i] + part[first + 1][i];
    for (int w = 2; w < segw; w += 2) v += part[first + w][i] + part[first + w + 1][i];
    return v;
}

template <typename XT>
__device__ __forceinline__ void load_x32(const XT* x, int64_t k0, int64_t n, float (&xf)[32]) {
    if (k0 + 32 <= n && (reinterpret_cast<uintptr_t>(x + k0) & 15) == 0) {
        if constexpr (sizeof(XT) == 2) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                union { uint4 u; __half h[8]; } pk;
                pk.u = reinterpret_cast<const uint4*>(x + k0)[q];
#pragma unroll
                for (int i = 0; i < 8; ++i) xf[8 * q + i] = __half2float(pk.h[i]);
            }
        } else {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const float4 f = reinterpret_cast<const float4*>(x + k0)[q];
                xf[4 * q] = f.x; xf[4 * q + 1] = f.y; xf[4 * q + 2] = f.z; xf[4 * q + 3] = f.w;
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < 32; ++i) {
            float v = 0.f;
            if (k0 + i < n) {
                if constexpr (sizeof(XT) == 2) v = __half2float(x[k0 + i]);
                else v = x[k0 + i];
            }
            xf[i] = v;                       // columns past n contribute nothing
        }
    }
}

// GSUB = number of grids inside a lane's 32 columns: 1 (one grid per row, or groups of a multiple of 32), 2 (16), 4 (8)
template <int BITS, int GSUB, int WAVES, typename XT>
__global__ __launch_bounds__(64 * WAVES) void matvec_kernel(PackedArgs a, const XT* x, float* y) {
    __shared__ float part[WAVES][MV_ROWS];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int groups = (int)(blockDim.x >> 6) >> a.segshift, grp = wave >> a.segshift, sw = wave & (a.segw - 1);
    const int64_t nseg = (a.n + MV_SEG - 1) / MV_SEG;
    constexpr int GL = 32 / GSUB;            // columns per grid inside the lane's 32
    const int64_t row_end = min(((int64_t)blockIdx.x + 1) * a.rows_per_wg, a.r);
    for (int64_t wg0 = (int64_t)blockIdx.x * a.rows_per_wg; wg0 < row_end; wg0 += groups * MV_ROWS) {
    const int64_t row0 = wg0 + grp * MV_ROWS;
    float acc[MV_ROWS];
#pragma unroll
    for (int rr = 0; rr < MV_ROWS; ++rr) acc[rr] = 0.f;
    for (int64_t s = sw; s < nseg; s += a.segw) {
        const int64_t k0 = s * MV_SEG + (int64_t)lane * 32;
        if (k0 >= a.n) continue;
        float xf[32];
        load_x32<XT>(x, k0, a.n, xf);
        float sx[GSUB];
#pragma unroll
        for (int j = 0; j < GSUB; ++j) {
            float t = 0.f;
#pragma unroll
            for (int i = 0; i < GL; ++i) t += xf[j * GL + i];
            sx[j] = t;
        }
        const int64_t w0 = (k0 >> 5) * BITS;
        const int64_t g0 = a.group ? k0 / a.group : 0;
#pragma unroll
        for (int rr = 0; rr < MV_ROWS; ++rr) {
            const int64_t row = min(row0 + rr, a.r - 1);         // rows past r repeat the last one and are dropped below
            const uint32_t* p = a.words + row * a.ldp + w0;
            uint32_t w[BITS];
#pragma unroll
            for (int i = 0; i < BITS; ++i) w[i] = (w0 + i < a.words_per_row) ? p[i] : 0u;
#pragma unroll
            for (int j = 0; j < GSUB; ++j) {
                float dot = 0.f;
#pragma unroll
                for (int i = 0; i < GL; ++i) dot = fmaf((float)code_at<BITS>(w, j * GL + i), xf[j * GL + i], dot);
                const int64_t gi = row * a.ngroups + min(g0 + j, a.ngroups - 1);
                acc[rr] = fmaf(a.scales[gi], dot - (float)a.zeros[gi] * sx[j], acc[rr]);
            }
        }
    }
    const float v = wave_sum4(acc[0], acc[1], acc[2], acc[3]);
    if ((lane & 15) == 0) part[wave][wave_sum_index(lane)] = v;
    __syncthreads();
    const int64_t row = wg0 + threadIdx.x;
    if (threadIdx.x < groups * MV_ROWS && row < a.r) y[row] = sum_parts<MV_ROWS>(part, (int)(threadIdx.x / MV_ROWS) * a.segw, a.segw, threadIdx.x % MV_ROWS);
    __syncthreads();
    }
}

// float16 vector, one grid per lane segment (one grid per row, or groups of a multiple of 32): two weights per
// v_dot2_f32_f16 on the pairs of halves 2^b + code made as above; the vector's halves are paired the same way once
// per segment.  The dot products accumulate sum (2^b + code) x in float32, and
// sum (code - zero) x = that - (2^b + zero) sum x;  the offset is of the size of the codes themselves, so the
// subtraction costs no accuracy worth naming.
constexpr int MV2_HALF = 4;      // rows of a wavefront are read four at a time: four or eight (NH = 1, 2) per step

// The b words of this lane's 32 columns for four consecutive rows (rows past r repeat the last one).  n is a multiple
// of 32 here, so a lane's words are all inside the row or all outside; `w0` is clamped by the caller for the latter,
// whose vector entries are zero.
template <int BITS>
__device__ __forceinline__ void mv_load_rows(uint32_t (&w)[MV2_HALF][BITS + 1], const PackedArgs& a, int rowbase, uint32_t w0) {
#pragma unroll
    for (int rr = 0; rr < MV2_HALF; ++rr) {
        // the row is the same for the whole wavefront: its address stays in scalar registers and the load takes the
        // lane's word offset as a 32-bit index (r and the words of a row fit 31 bits, checked on the host)
        const int row = __builtin_amdgcn_readfirstlane(min(rowbase + rr, (int)a.r - 1));
        const uint32_t* prow = a.words + (int64_t)row * a.ldp;
        struct __attribute__((packed, aligned(4))) Words { uint32_t v[BITS]; };
        const Words t = *reinterpret_cast<const Words*>(reinterpret_cast<const char*>(prow) + w0 * 4u);      // one load of b words
#pragma unroll
        for (int i = 0; i < BITS; ++i) w[rr][i] = t.v[i];
        w[rr][BITS] = 0u;
    }
}

// The same two instructions as volatile statements: they keep their program order, so a pair of halves is consumed by
// its dot product right after it is made.  Left to itself the scheduler makes all 64 pairs of four rows first and
// holds them in registers, which costs a wavefront per SIMD.
__device__ __forceinline__ uint32_t and_or_ordered(uint32_t a, uint32_t mask, uint32_t c) {
    uint32_t v;
    asm volatile("v_and_or_b32 %0, %1, %2, %3" : "=v"(v) : "v"(a), "s"(mask), "v"(c));
    return v;
}
__device__ __forceinline__ void dot2_ordered(float& d, uint32_t pair, half2v xv) {
    asm volatile("v_dot2_f32_f16 %0, %1, %2, %0" : "+v"(d) : "v"(pair), "v"(xv));
}

// Scale and zero point of four rows at the lane's group
struct MvGrid { float sc[MV2_HALF]; int zr[MV2_HALF]; };
__device__ __forceinline__ void mv_load_grid(MvGrid& gr, const PackedArgs& a, int rowbase, uint32_t g0) {
#pragma unroll
    for (int rr = 0; rr < MV2_HALF; ++rr) {
        const int row = __builtin_amdgcn_readfirstlane(min(rowbase + rr, (int)a.r - 1));
        const int64_t gbase = (int64_t)row * a.ngroups;      // scalar; the lane's group is a 32-bit index on top
        gr.sc[rr] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(a.scales + gbase) + g0 * 4u);
        gr.zr[rr] = *reinterpret_cast<const int32_t*>(reinterpret_cast<const char*>(a.zeros + gbase) + g0 * 4u);
    }
}

// acc[rr] += scale * (sum (2^b + code) x - (2^b + zero) sum x) over this lane's 32 columns, for four rows
template <int BITS>
__device__ __forceinline__ void mv_dot_rows(const uint32_t (&w)[MV2_HALF][BITS + 1], const half2v (&xq)[16], float sx, float* acc, const MvGrid& gr) {
    constexpr int WANT = 10 - BITS;
    constexpr uint32_t M = (1u << BITS) - 1u;
    constexpr uint32_t MASK_LO = M << WANT, MASK_HI = M << (16 + WANT), MASK = MASK_LO | MASK_HI;
    const uint32_t magic = 0x3C003C00u + (uint32_t)BITS * 0x04000400u;       // (2^b, 2^b) as two halves
    const float offset = (float)(1 << BITS);
#pragma unroll
    for (int rr = 0; rr < MV2_HALF; ++rr) {
        // two interleaved chains per row, so consecutive dot products do not wait for each other
        float d0 = 0.f, d1 = 0.f;
        uint32_t joined[3] = {0u, 0u, 0u};
        if constexpr (BITS == 3) {
            joined[0] = __builtin_amdgcn_perm(w[rr][1], w[rr][0], 0x07060100u);      // low half of w0, high half of w1
            joined[1] = __builtin_amdgcn_perm(w[rr][0], w[rr][2], 0x07060100u);      // low half of w2, high half of w0
            joined[2] = __builtin_amdgcn_perm(w[rr][2], w[rr][1], 0x07060100u);      // low half of w1, high half of w2
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const PairSpec sp = PairTable<BITS>::at(i);
            uint32_t v;
            if (sp.lo_word < 0) {
                const uint32_t ta = stream_bits<BITS>(w[rr], BITS * sp.k_lo - WANT);
                const uint32_t tb = stream_bits<BITS>(w[rr], BITS * sp.k_hi - (16 + WANT));
                v = and_or_ordered(tb, MASK_HI, and_or_ordered(ta, MASK_LO, magic));
            } else {
                uint32_t m;
                if (sp.lo_word == sp.hi_word) m = w[rr][sp.lo_word];
                else m = joined[sp.lo_word == 0 ? 0 : (sp.lo_word == 2 ? 1 : 2)];
                const uint32_t t = sp.rel >= WANT ? (m >> (sp.rel - WANT)) : (m << (WANT - sp.rel));
                v = and_or_ordered(t, MASK, magic);
            }
            if (i & 1) dot2_ordered(d1, v, xq[i]);
            else       dot2_ordered(d0, v, xq[i]);
        }
        // a dot product's result wants three wait states before another kind of instruction reads it; inside a statement the
        // compiler does not see the one that wrote it
        asm volatile("s_nop 3" : "+v"(d0), "+v"(d1));
        acc[rr] = fmaf(gr.sc[rr], (d0 + d1) - (offset + (float)gr.zr[rr]) * sx, acc[rr]);
    }
}

// The words of the next four rows are requested before the current four are multiplied (within a segment, and across to
// the wavefront's next segment), so a wavefront always has loads in flight while it computes.
// NH: halves of four rows per step.  With eight rows a vector entry's preparation serves twice as many; with four there are twice as many
// wavefronts, and up to 16 of them in a workgroup (mv_plan).

// The lane's 32 vector entries, two halves per register, zeros past n, then paired like the codes; returns their sum on top of sx
__device__ __forceinline__ void mv_load_x(uint32_t (&xp)[16], const __half* x, int64_t k0, int64_t n) {
    const bool inside = k0 < n;
    const __half* xsrc = x + min(k0, n - 32);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint4 u = reinterpret_cast<const uint4*>(xsrc)[q];
        xp[4 * q] = inside ? u.x : 0u; xp[4 * q + 1] = inside ? u.y : 0u; xp[4 * q + 2] = inside ? u.z : 0u; xp[4 * q + 3] = inside ? u.w : 0u;
    }
}
template <int BITS>
__device__ __forceinline__ float mv_pair_x(half2v (&xq)[16], const uint32_t (&xp)[16], float sx) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        sx = __builtin_amdgcn_fdot2(__builtin_bit_cast(half2v, xp[i]), __builtin_bit_cast(half2v, 0x3C003C00u), sx, false);
        const PairSpec sp = PairTable<BITS>::at(i);
        const uint32_t lo = (xp[sp.k_lo >> 1] >> (16 * (sp.k_lo & 1))) & 0xFFFFu;
        const uint32_t hi = (sp.k_hi & 1) ? (xp[sp.k_hi >> 1] & 0xFFFF0000u) : (xp[sp.k_hi >> 1] << 16);
        xq[i] = __builtin_bit_cast(half2v, lo | hi);
    }
    return sx;
}

template <int BITS, int NH, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void matvec_dot2_kernel(PackedArgs a, const __half* x, float* y) {
    constexpr int ROWS = NH * MV2_HALF;
    __shared__ float part[WAVES][ROWS];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int groups = (int)(blockDim.x >> 6) >> a.segshift, grp = wave >> a.segshift, sw = wave & (a.segw - 1);
    const int64_t nseg = (a.n + MV_SEG - 1) / MV_SEG;
    const int64_t row_end = min(((int64_t)blockIdx.x + 1) * a.rows_per_wg, a.r);
    const uint32_t wlast = (uint32_t)(a.words_per_row - BITS);      // n is a multiple of 32 and at least 32
    auto words_at = [&](int64_t seg) { return min((uint32_t)(((seg * MV_SEG) >> 5) + lane) * BITS, wlast); };
    for (int64_t wg0 = (int64_t)blockIdx.x * a.rows_per_wg; wg0 < row_end; wg0 += groups * ROWS) {
    float acc[ROWS];
#pragma unroll
    for (int rr = 0; rr < ROWS; ++rr) acc[rr] = 0.f;
    uint32_t wa[MV2_HALF][BITS + 1], wb[MV2_HALF][BITS + 1];
    const int row0i = (int)wg0 + grp * ROWS;
    if (sw < nseg) mv_load_rows<BITS>(wa, a, row0i, words_at(sw));
#pragma unroll 1
    for (int64_t s = sw; s < nseg; s += a.segw) {
        const int64_t k0 = s * MV_SEG + (int64_t)lane * 32;      // lanes past the last column: any words, zero vector entries
        if constexpr (NH == 2) mv_load_rows<BITS>(wb, a, row0i + MV2_HALF, words_at(s));
        uint32_t xp[16];
        mv_load_x(xp, x, k0, a.n);
        // column / group size without the 64-bit division (n < 2^31 is checked on the host)
        const uint32_t kc = (uint32_t)min(k0, a.n - 32);
        const uint32_t g0 = a.group == 0 ? 0u : (a.gshift >= 0 ? kc >> a.gshift : kc / (uint32_t)a.group);
        MvGrid gr;
        mv_load_grid(gr, a, row0i, g0);
        if constexpr (NH == 1)
            if (s + a.segw < nseg) mv_load_rows<BITS>(wb, a, row0i, words_at(s + a.segw));
        asm volatile("" ::: "memory");                       // the requests above stay above the arithmetic below
        half2v xq[16];
        const float sx = mv_pair_x<BITS>(xq, xp, 0.f);
        mv_dot_rows<BITS>(wa, xq, sx, acc, gr);
        if constexpr (NH == 2) {
            mv_load_grid(gr, a, row0i + MV2_HALF, g0);
            if (s + a.segw < nseg) mv_load_rows<BITS>(wa, a, row0i, words_at(s + a.segw));
            asm volatile("" ::: "memory");
            mv_dot_rows<BITS>(wb, xq, sx, acc + MV2_HALF, gr);
        } else {
#pragma unroll
            for (int rr = 0; rr < MV2_HALF; ++rr)
#pragma unroll
                for (int i = 0; i <= BITS; ++i) wa[rr][i] = wb[rr][i];
        }
    }
#pragma unroll
    for (int h = 0; h < NH; ++h) {
        const float v = wave_sum4(acc[4 * h], acc[4 * h + 1], acc[4 * h + 2], acc[4 * h + 3]);
        if ((lane & 15) == 0) part[wave][4 * h + wave_sum_index(lane)] = v;
    }
    __syncthreads();
    const int64_t row = wg0 + threadIdx.x;
    if (threadIdx.x < groups * ROWS && row < a.r) y[row] = sum_parts<ROWS>(part, (int)(threadIdx.x / ROWS) * a.segw, a.segw, threadIdx.x % ROWS);
    __syncthreads();
    }
}

// ---- one grid per row: the dot products on the matrix cores --------------------------------------------------------
// Same loads, same pairs of halves, but the pairs are not multiplied by v_dot2: two pair registers (4 weights) are the A
// operand and the two matching registers of the vector the B operand of one v_mfma_f32_16x16x16_f16.  The instruction
// computes D[i][j] += sum over the four lanes kb of <weights of lane (i, kb), vector entries of lane (j, kb)>
// (lane = i + 16 kb on the A side, j + 16 kb on the B side), so its DIAGONAL accumulates exactly the dot products the
// lanes want -- every lane's weights with its own vector entries, summed over four lanes at a time -- and the other 240
// entries (one lane's weights with another lane's entries) are never read.  That takes a third of the vector
// instructions off the path that bounds the kernel, at 8 matrix-core instructions per row and segment, which run beside
// the unpacking of other wavefronts.  With one grid per row the scale, the zero point and the 2^b offset come in at the
// very end:  y = scale (sum (2^b + code) x - (2^b + zero) sum x).
typedef _Float16 half4v __attribute__((ext_vector_type(4)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));

// codes_as_half_pairs with the and-or written in C: what feeds a matrix-core instruction must be an instruction the
// compiler knows, so that it can keep the wait states the hardware wants between a vector write and the matrix read of
// the same register (an inline-assembly statement hides its instruction from that check).
template <int BITS>
__device__ __forceinline__ void codes_as_half_pairs_plain(const uint32_t (&w)[BITS + 1], uint32_t (&pr)[16]) {
    constexpr int WANT = 10 - BITS;
    constexpr uint32_t M = (1u << BITS) - 1u;
    constexpr uint32_t MASK_LO = M << WANT, MASK_HI = M << (16 + WANT), MASK = MASK_LO | MASK_HI;
    uint32_t magic = 0x3C003C00u + (uint32_t)BITS * 0x04000400u;             // (2^b, 2^b) as two halves
    // the constants in registers whose contents the compiler does not know: v_and_or_b32 takes no literals here, and with
    // known constants the compiler prefers an and and an or with one literal each
    uint32_t mask = MASK, mask_lo = MASK_LO, mask_hi = MASK_HI;
    asm volatile("" : "+s"(mask), "+s"(mask_lo), "+s"(mask_hi), "+v"(magic));
    uint32_t joined[3] = {0u, 0u, 0u};
    if constexpr (BITS == 3) {
        joined[0] = __builtin_amdgcn_perm(w[1], w[0], 0x07060100u);      // low half of w0, high half of w1
        joined[1] = __builtin_amdgcn_perm(w[0], w[2], 0x07060100u);      // low half of w2, high half of w0
        joined[2] = __builtin_amdgcn_perm(w[2], w[1], 0x07060100u);      // low half of w1, high half of w2
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const PairSpec sp = PairTable<BITS>::at(i);
        if (sp.lo_word < 0) {
            const uint32_t ta = stream_bits<BITS>(w, BITS * sp.k_lo - WANT);
            const uint32_t tb = stream_bits<BITS>(w, BITS * sp.k_hi - (16 + WANT));
            pr[i] = (tb & mask_hi) | ((ta & mask_lo) | magic);
        } else {
            uint32_t m;
            if (sp.lo_word == sp.hi_word) m = w[sp.lo_word];
            else m = joined[sp.lo_word == 0 ? 0 : (sp.lo_word == 2 ? 1 : 2)];
            const uint32_t t = sp.rel >= WANT ? (m >> (sp.rel - WANT)) : (m << (WANT - sp.rel));
            pr[i] = (t & mask) | magic;
        }
    }
}

template <int BITS>
__device__ __forceinline__ void mv_mfma_rows(const uint32_t (&w)[MV2_HALF][BITS + 1], const half2v (&xq)[16], float4v* acc) {
#pragma unroll
    for (int rr = 0; rr < MV2_HALF; ++rr) {
        uint32_t pr[16];
        codes_as_half_pairs_plain<BITS>(w[rr], pr);
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const u32x2v av = {pr[2 * t], pr[2 * t + 1]};
            const u32x2v bv = {__builtin_bit_cast(uint32_t, xq[2 * t]), __builtin_bit_cast(uint32_t, xq[2 * t + 1])};
            acc[rr] = __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(half4v, av), __builtin_bit_cast(half4v, bv), acc[rr], 0, 0, 0);
        }
    }
}

template <int BITS, int NH, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void matvec_mfma_kernel(PackedArgs a, const __half* x, float* y) {
    constexpr int ROWS = NH * MV2_HALF;
    __shared__ float part[WAVES][ROWS + 1];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int groups = (int)(blockDim.x >> 6) >> a.segshift, grp = wave >> a.segshift, sw = wave & (a.segw - 1);
    const int64_t nseg = (a.n + MV_SEG - 1) / MV_SEG;
    const int64_t row_end = min(((int64_t)blockIdx.x + 1) * a.rows_per_wg, a.r);
    // this lane's element of the diagonal of D: lane = j + 16 ib holds D[4 ib + e][j], e = 0 .. 3
    const int dj = lane & 15, dib = lane >> 4;
    const bool on_diag = (dj >> 2) == dib;
    const int de = dj & 3;
    const uint32_t wlast = (uint32_t)(a.words_per_row - BITS);      // n is a multiple of 32 and at least 32
    auto words_at = [&](int64_t seg) { return min((uint32_t)(((seg * MV_SEG) >> 5) + lane) * BITS, wlast); };
    for (int64_t wg0 = (int64_t)blockIdx.x * a.rows_per_wg; wg0 < row_end; wg0 += groups * ROWS) {
    float4v acc[ROWS];
#pragma unroll
    for (int rr = 0; rr < ROWS; ++rr) acc[rr] = float4v{0.f, 0.f, 0.f, 0.f};
    float sx = 0.f;                                          // sum of this lane's vector entries over its segments
    uint32_t wa[MV2_HALF][BITS + 1], wb[MV2_HALF][BITS + 1];
    const int row0i = (int)wg0 + grp * ROWS;
    if (sw < nseg) mv_load_rows<BITS>(wa, a, row0i, words_at(sw));
#pragma unroll 1
    for (int64_t s = sw; s < nseg; s += a.segw) {
        const int64_t k0 = s * MV_SEG + (int64_t)lane * 32;      // lanes past the last column: any words, zero vector entries
        if constexpr (NH == 2) mv_load_rows<BITS>(wb, a, row0i + MV2_HALF, words_at(s));
        uint32_t xp[16];
        mv_load_x(xp, x, k0, a.n);
        if constexpr (NH == 1)
            if (s + a.segw < nseg) mv_load_rows<BITS>(wb, a, row0i, words_at(s + a.segw));
        asm volatile("" ::: "memory");                       // the requests above stay above the arithmetic below
        half2v xq[16];
        sx = mv_pair_x<BITS>(xq, xp, sx);
        mv_mfma_rows<BITS>(wa, xq, acc);
        if constexpr (NH == 2) {
            if (s + a.segw < nseg) mv_load_rows<BITS>(wa, a, row0i, words_at(s + a.segw));
            asm volatile("" ::: "memory");
            mv_mfma_rows<BITS>(wb, xq, acc + MV2_HALF);
        } else {
#pragma unroll
            for (int rr = 0; rr < MV2_HALF; ++rr)
#pragma unroll
                for (int i = 0; i <= BITS; ++i) wa[rr][i] = wb[rr][i];
        }
    }
#pragma unroll
    for (int h = 0; h < NH; ++h) {
        float d[4];
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            const float4v c = acc[4 * h + rr];
            const float e = de == 0 ? c.x : (de == 1 ? c.y : (de == 2 ? c.z : c.w));
            d[rr] = on_diag ? e : 0.f;
        }
        const float v = wave_sum4(d[0], d[1], d[2], d[3]);
        if ((lane & 15) == 0) part[wave][4 * h + wave_sum_index(lane)] = v;
    }
    const float sxs = wave_sum4(sx, 0.f, 0.f, 0.f);
    if (lane == 0) part[wave][ROWS] = sxs;
    __syncthreads();
    const int64_t row = wg0 + threadIdx.x;
    if (threadIdx.x < groups * ROWS && row < a.r) {
        const int first = (int)(threadIdx.x / ROWS) * a.segw;
        const float dots = sum_parts<ROWS + 1>(part, first, a.segw, threadIdx.x % ROWS), sum = sum_parts<ROWS + 1>(part, first, a.segw, ROWS);
        y[row] = a.scales[row * a.ngroups] * (dots - ((float)(1 << BITS) + (float)a.zeros[row * a.ngroups]) * sum);
    }
    __syncthreads();
    }
}

__global__ void zero_vector_kernel(float* y, int64_t r) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < r) y[i] = 0.f;
}

static int check_packed(const char* who, const uint32_t* words, int64_t ldp, int64_t r, int64_t n, int bits,
                        const float* scales, const int32_t* zeros, int64_t group, PackedArgs* a) {
    if (r < 0 || n < 0) return fail(GPTQ_ERR_INVALID_ARG, "%s: negative size", who);
    if (bits < 2 || bits > 4) return fail(GPTQ_ERR_INVALID_ARG, "%s: bits must be 2, 3 or 4 (got %d)", who, bits);
    if (group < 0) return fail(GPTQ_ERR_INVALID_ARG, "%s: negative group", who);
    if (group > 0 && n % group) return fail(GPTQ_ERR_INVALID_ARG, "%s: n must be a multiple of the group size", who);
    if (r == 0 || n == 0) return GPTQ_OK;
    if (!words || !scales || !zeros) return fail(GPTQ_ERR_INVALID_ARG, "%s: null pointer", who);
    const int64_t wpr = (n * bits + 31) / 32;
    if (ldp < wpr) return fail(GPTQ_ERR_INVALID_ARG, "%s: word pitch smaller than ceil(n*bits/32)", who);
    a->words = words; a->ldp = ldp; a->r = r; a->n = n; a->words_per_row = wpr;
    a->scales = scales; a->zeros = zeros; a->group = group; a->ngroups = group ? n / group : 1;
    a->gshift = -1;
    if (group > 0 && (group & (group - 1)) == 0) { int sh = 0; while (((int64_t)1 << sh) < group) ++sh; a->gshift = sh; }
    return -1;
}

}  // namespace gptq

using namespace gptq;

extern "C" int gptq_dequantize_packed(const uint32_t* words, int64_t ldp, int64_t r, int64_t n, int bits,
                                      const float* scales, const int32_t* zeros, int64_t group,
                                      void* out, int odtype, int64_t ldo, void* stream) {
    PackedArgs a{};
    const int rc = check_packed("dequantize_packed", words, ldp, r, n, bits, scales, zeros, group, &a);
    if (rc >= 0) return rc;
    if (odtype != GPTQ_F16 && odtype != GPTQ_F32) return fail(GPTQ_ERR_INVALID_ARG, "dequantize_packed: output type must be float16 or float32");
    if (!out) return fail(GPTQ_ERR_INVALID_ARG, "dequantize_packed: null pointer");
    if (ldo < n) return fail(GPTQ_ERR_INVALID_ARG, "dequantize_packed: ldo < n");
    hipStream_t s = static_cast<hipStream_t>(stream);
    const size_t osz = odtype == GPTQ_F16 ? 2 : 4;
    if (n % 8 == 0 && n < 0x7fffffffLL && (group == 0 || group % 8 == 0) && aligned(out, 16) && (ldo * osz) % 16 == 0) {
        const int64_t octets = n / 8;
        const dim3 grid((unsigned)std::min<int64_t>(r, 256 * 64));
#define GPTQ_DQ8(B)                                                                                                              \
        if (odtype == GPTQ_F16) hipLaunchKernelGGL((dequantize8_kernel<B, _Float16>), grid, dim3(256), 0, s, a, static_cast<_Float16*>(out), ldo, octets); \
        else hipLaunchKernelGGL((dequantize8_kernel<B, float>), grid, dim3(256), 0, s, a, static_cast<float*>(out), ldo, octets)
        if (bits == 2) { GPTQ_DQ8(2); } else if (bits == 3) { GPTQ_DQ8(3); } else { GPTQ_DQ8(4); }
#undef GPTQ_DQ8
        GPTQ_LAUNCH_CHECK();
        return GPTQ_OK;
    }
    const int64_t g32 = (n + 7) / 8;               // octets of codes per row
    if (r * g32 > (int64_t)0x7fffffff * 256) return fail(GPTQ_ERR_UNSUPPORTED, "dequantize_packed: too large");
    const unsigned blocks = (unsigned)ceil_div(r * g32, 256);
#define GPTQ_DQ(B)                                                                                                              \
    if (odtype == GPTQ_F16) hipLaunchKernelGGL((dequantize_kernel<B, __half>), dim3(blocks), dim3(256), 0, s, a, static_cast<__half*>(out), ldo, g32); \
    else hipLaunchKernelGGL((dequantize_kernel<B, float>), dim3(blocks), dim3(256), 0, s, a, static_cast<float*>(out), ldo, g32)
    if (bits == 2) { GPTQ_DQ(2); } else if (bits == 3) { GPTQ_DQ(3); } else { GPTQ_DQ(4); }
#undef GPTQ_DQ
    GPTQ_LAUNCH_CHECK();
    return GPTQ_OK;
}

// CUs of the current device, asked for once per device; several threads may ask at a time.
static int64_t chip_cus() {
    constexpr int MAXDEV = 64, USUAL = 256;
    static std::atomic<int> known[MAXDEV];
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAXDEV) return USUAL;
    if ((cus = known[dev].load(std::memory_order_relaxed)) > 0) return cus;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) return USUAL;
    known[dev].store(cus, std::memory_order_relaxed);
    return cus;
}

// How a matrix is dealt out: the rows a wavefront takes at a time (4 NH), the wavefronts that share a row (segw, each every segw-th segment of
// 2048 columns) and those of a workgroup.  Where rows have fewer segments than a workgroup has wavefronts these take other rows (before,
// they had nothing to do); few rows of many segments are shared by up to 16; and a workgroup is smaller where there would be
// fewer than CUs.  Measured, us per launch in a graph, 3 bits with one grid per row, four wavefronts a row and eight rows throughout as
// before / now: 256 x 256 5.0 / 3.0, 4096 x 4096 6.2 / 4.0, 49152 x 256 25.9 / 9.5, 49152 x 4096 35.5 / 19.5, 256 x 49152 10.9 / 6.6 (4 bits,
// groups of 128: 4.8 / 2.8, 6.0 / 3.7, 23.7 / 9.3, 35.9 / 22.1, 13.2 / 6.0).
// Four rows at a time up to one segment of them for each of the 3072 wavefronts that hide a launch's latency (12288 x 2048 4.5 / 5.0 with eight,
// 2048 x 12288 5.5 / 5.4, 8192 x 4096 5.3 / 5.1) and up to 1024 rows, where 16 wavefronts of a workgroup share them (1024 x 49152
// 7.1 / 9.1; 1500 12.8 / 9.9); beyond, eight, which prepare a vector entry for twice the weights, shared by 8 up to 4096 rows
// (1500 x 49152 9.9 / 11.5 with 4, 4000 x 24576 9.8 / 10.4, 12288 x 12288 20.3 / 16.7).  The general kernel takes four: with 16
// wavefronts 1024 x 49152 14.6 -> 11.6, from 1500 rows on nothing or a loss.
struct MvPlan { int nh, waves, segw; int64_t rows_per_wg; unsigned blocks; };
static MvPlan mv_plan(int64_t r, int64_t n, bool may_take_eight) {
    const int64_t nseg = ceil_div(n, MV_SEG);
    const bool few = r <= 1024;
    int nh = may_take_eight && !few && ceil_div(r, 4) * nseg > 3072 ? 2 : 1;
    int most = few ? MV_MAX_WAVES : !may_take_eight ? 4 : nh == 1 ? MV_MAX_WAVES : r <= 4096 ? 8 : 4;
    const int64_t cus = chip_cus();
    MvPlan p{};
    p.nh = nh;
    p.segw = 1;
    while (p.segw < most && p.segw < nseg) p.segw *= 2;
    p.waves = p.segw < 4 ? 4 : p.segw;
    while (p.waves > p.segw && ceil_div(r, p.waves / p.segw * 4 * p.nh) < cus) p.waves /= 2;      // a workgroup for every CU
    const int chunk = p.waves / p.segw * 4 * p.nh;
    p.rows_per_wg = (int64_t)round_up((size_t)ceil_div(r, std::max<int64_t>(1, cus * 32 / p.waves)), (size_t)chunk);
    p.blocks = (unsigned)ceil_div(r, p.rows_per_wg);
    return p;
}

template <int BITS, typename XT>
static void launch_matvec(PackedArgs a, const XT* x, float* y, hipStream_t s) {
    const int gsub = (a.group == 0 || a.group % 32 == 0) ? 1 : (int)(32 / a.group);
    if constexpr (sizeof(XT) == 2) {
        // the fast kernel wants whole lanes (32 columns each) and 16-byte loads of the vector
        if (gsub == 1 && a.n % 32 == 0 && a.n >= 32 && a.n < 0x7fffffffLL && a.r < 0x7fffff00LL && a.words_per_row < 0x3fffffffLL &&
            a.ngroups < 0x3fffffffLL && (reinterpret_cast<uintptr_t>(x) & 15) == 0) {
            const MvPlan p = mv_plan(a.r, a.n, true);
            a.rows_per_wg = p.rows_per_wg; a.segw = p.segw; a.segshift = __builtin_ctz(p.segw);
            const dim3 grid(p.blocks), block(64 * p.waves);
#define GPTQ_MV2(K)                                                                                             \
            if (p.nh == 1) hipLaunchKernelGGL((K<BITS, 1, MV_MAX_WAVES>), grid, block, 0, s, a, x, y);          \
            else if (p.waves > 4) hipLaunchKernelGGL((K<BITS, 2, MV_MAX_WAVES>), grid, block, 0, s, a, x, y);   \
            else hipLaunchKernelGGL((K<BITS, 2, 4>), grid, block, 0, s, a, x, y)
            if (a.group == 0) { GPTQ_MV2(matvec_mfma_kernel); } else { GPTQ_MV2(matvec_dot2_kernel); }
#undef GPTQ_MV2
            return;
        }
    }
    const MvPlan p = mv_plan(a.r, a.n, false);
    a.rows_per_wg = p.rows_per_wg; a.segw = p.segw; a.segshift = __builtin_ctz(p.segw);
    const dim3 grid(p.blocks), block(64 * p.waves);
#define GPTQ_MV1(G)                                                                                             \
    if (p.waves > 4) hipLaunchKernelGGL((matvec_kernel<BITS, G, MV_MAX_WAVES, XT>), grid, block, 0, s, a, x, y); \
    else hipLaunchKernelGGL((matvec_kernel<BITS, G, 4, XT>), grid, block, 0, s, a, x, y)
    if (gsub == 1) { GPTQ_MV1(1); } else if (gsub == 2) { GPTQ_MV1(2); } else { GPTQ_MV1(4); }
#undef GPTQ_MV1
}

extern "C" int gptq_matvec_packed(const uint32_t* words, int64_t ldp, int64_t r, int64_t n, int bits,
                                  const float* scales, const int32_t* zeros, int64_t group,
                                  const void* x, int xdtype, float* y, void* stream) {
    PackedArgs a{};
    const int rc = check_packed("matvec_packed", words, ldp, r, n, bits, scales, zeros, group, &a);
    if (rc >= 0) {
        if (rc == GPTQ_OK && r > 0 && n == 0) {          // an empty sum: y = 0
            if (!y) return fail(GPTQ_ERR_INVALID_ARG, "matvec_packed: null pointer");
            hipLaunchKernelGGL(zero_vector_kernel, dim3((unsigned)ceil_div(r, 256)), dim3(256), 0, static_cast<hipStream_t>(stream), y, r);
            GPTQ_LAUNCH_CHECK();
        }
        return rc;
    }
    if (xdtype != GPTQ_F16 && xdtype != GPTQ_F32) return fail(GPTQ_ERR_INVALID_ARG, "matvec_packed: vector type must be float16 or float32");
    if (!x || !y) return fail(GPTQ_ERR_INVALID_ARG, "matvec_packed: null pointer");
    if (group > 0 && group % 32 && group != 8 && group != 16)
        return fail(GPTQ_ERR_UNSUPPORTED, "matvec_packed: group size %lld not built (8, 16 or a multiple of 32)", (long long)group);
    if (ceil_div(r, MV_ROWS) > 0x7fffffffLL) return fail(GPTQ_ERR_UNSUPPORTED, "matvec_packed: too many rows");
    hipStream_t s = static_cast<hipStream_t>(stream);
#define GPTQ_MV(B)                                                                              \
    if (xdtype == GPTQ_F16) launch_matvec<B, __half>(a, static_cast<const __half*>(x), y, s);   \
    else launch_matvec<B, float>(a, static_cast<const float*>(x), y, s)
    if (bits == 2) { GPTQ_MV(2); } else if (bits == 3) { GPTQ_MV(3); } else { GPTQ_MV(4); }
#undef GPTQ_MV
    GPTQ_LAUNCH_CHECK();
    return GPTQ_OK;
}
