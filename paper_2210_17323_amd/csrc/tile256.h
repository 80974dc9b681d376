// One step of a 256 x 256 tile by four wavefronts of 128 x 128, 16-bit operands in LDS, 256 float32 accumulators a lane: what the
// Hessian's kernel does between two barriers.  Its instructions and how its results leave are those of the split products too.
//
// Bound by the power the matrix cores may draw, which sets the clock.  A 32x32x16 instruction reads and writes four times the
// accumulators of a 16x16x32 one for twice the products; a loop of registers holds, on normal data, 1600 TFLOP/s (float16) and 1740
// (bfloat16) with the larger shape and 1870 and 2005 with the smaller (60 % zeros 2040 / 2350, all zeros 2480 either way).  Both add 8
// products at a time to the accumulator, k ascending: the same bits.  Whole kernels: a Hessian launch of 49152 channels x 32768 tokens behind
// a ReLU 55.5 -> 49.4 ms, 12288 x 32768 normal 4.86 -> 4.25 (matrix cores busy 67 -> 74 % of the cycles, 1.48 -> 1.54 GHz).
#pragma once
#include "common.h"

namespace gptq {

typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

// c += a b, the accumulator in place.  As a statement of its own and not the builtin: with 256 accumulator registers in groups of
// four the compiler gives the builtin's result another place than its addend and copies and spills between them.  What it
// cannot see is that this is a matrix-core instruction: the callers see to it that no vector instruction writes an operand
// right before, and wait before the first read of an accumulator (mfma_settle); tests/test_matrix_instruction_waits.py looks for both in
// the assembly.
template <bool IS_BF16>
__device__ __forceinline__ void mfma16x16_acc(floatx4& c, uint4 a, uint4 b) {
    if constexpr (IS_BF16)
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(__builtin_bit_cast(bf16x8, a)), "v"(__builtin_bit_cast(bf16x8, b)));
    else
        asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(c) : "v"(__builtin_bit_cast(halfx8, a)), "v"(__builtin_bit_cast(halfx8, b)));
}
// The last results of a loop of these, four at a time, before something else reads them: 16 wait states and more.
__device__ __forceinline__ void mfma_settle(floatx4& a, floatx4& b, floatx4& c, floatx4& d) {
    asm volatile("s_nop 15\n\ts_nop 3" : "+a"(a), "+a"(b), "+a"(c), "+a"(d));
}

// Rows i, i + 4, i + 8, i + 12 of a 16 x 64 strip of results, four accumulators side by side, a row over the 64 lanes: 256 bytes in a row for
// the memory system, where the accumulators as they lie are four rows of 64.
__device__ __forceinline__ void mfma_rows64(const floatx4* acc, int i, float (&row)[4]) {
    uint32_t x[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = __float_as_uint(acc[q][i]);
    const auto a = __builtin_amdgcn_permlane16_swap(x[0], x[1], false, false);      // columns 0 .. 31: rows i and i + 8, i + 4 and i + 12
    const auto b = __builtin_amdgcn_permlane16_swap(x[2], x[3], false, false);      // columns 32 .. 63
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const auto c = __builtin_amdgcn_permlane32_swap(a[q], b[q], false, false);
        row[q] = __uint_as_float(c[0]);
        row[q + 2] = __uint_as_float(c[1]);
    }
}

// A stage holds a step of 32 k of both operands, A's panel of 256 rows and behind it B's: rows of 64 bytes, the 16-byte chunk c of
// row r at position c ^ ((r / 4) % 4), so that 16 consecutive rows, what 16 lanes of a 16-byte read touch together, fall on
// all 16 bank quads.
template <bool IS_BF16>
struct Tile256Lane {
    static constexpr int B_PANEL = 256 * 64;
    // acc[s][u]: rows wm*128 + s*16 + 4 (lane / 16) + 0..3, column wn*128 + u*16 + lane % 16
    floatx4 acc[8][8];
    uint4 fa[8], fb[8];
    int rowA, rowB;

    // This lane's operand rows are wm*128 + s*16 + lane%16 (A) and wn*128 + u*16 + lane%16 (B), its chunk lane/16: the
    // swizzle term is (lane / 4) % 4 for all of them, and s / u only add a constant 1024 bytes.
    __device__ __forceinline__ Tile256Lane(int lane, int wm, int wn) {
        const int l16 = lane & 15, chunk = ((lane >> 4) ^ ((l16 >> 2) & 3)) << 4;
        rowA = (wm * 128 + l16) * 64 + chunk;
        rowB = B_PANEL + (wn * 128 + l16) * 64 + chunk;
    }
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int s = 0; s < 8; ++s)
#pragma unroll
            for (int u = 0; u < 8; ++u)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[s][u][i] = 0.f;
    }
    __device__ __forceinline__ void fetchA(const unsigned char* st, int s) { fa[s] = *reinterpret_cast<const uint4*>(st + rowA + s * 1024); }
    __device__ __forceinline__ void fetchB(const unsigned char* st, int u) { fb[u] = *reinterpret_cast<const uint4*>(st + rowB + u * 1024); }
    __device__ __forceinline__ void fetch_first(const unsigned char* st) {
#pragma unroll
        for (int i = 0; i < 4; ++i) { fetchA(st, i); fetchB(st, i); }
    }
    // A quarter of the wavefront's tile, 64 x 64: rows 64 hs, columns 64 hu
    template <class Fetch, class Copy>
    __device__ __forceinline__ void quarter(int hs, int hu, Fetch&& fetch, Copy&& copy) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int s = 4 * hs + i;
#pragma unroll
            for (int j = 0; j < 4; ++j) {                // back and forth: one operand changes at a time (1 % of the power)
                const int u = 4 * hu + ((i & 1) ? 3 - j : j);
                mfma16x16_acc<IS_BF16>(acc[s][u], fa[s], fb[u]);
                if (i < 2 && (j & 1)) fetch(2 * i + (j >> 1));
                if ((i & 1) && j == 2) copy(i >> 1);
            }
        }
    }
    // One step out of `cur`.  The fragments of the first half of the rows and of the columns are there already; a quarter fetches what a
    // later one wants into the registers that are free by then -- the other rows, the other columns, then both first halves of the
    // NEXT step (`nxt`, whose copies have landed) --, eight MFMAs before they are read, so that none waits for an LDS round trip,
    // not even right after the barrier.  copy(0) .. copy(7) issue the step's copies, one every eight MFMAs: with one wavefront per SIMD
    // nothing else can issue while a copy instruction is being accepted (tens of cycles each).
    template <class Copy>
    __device__ __forceinline__ void multiply(const unsigned char* cur, const unsigned char* nxt, Copy&& copy) {
        quarter(0, 0, [&](int i) { fetchA(cur, 4 + i); }, [&](int i) { copy(i); });
        quarter(1, 0, [&](int i) { fetchB(cur, 4 + i); }, [&](int i) { copy(2 + i); });
        quarter(0, 1, [&](int i) { fetchB(nxt, i); }, [&](int i) { copy(4 + i); });
        quarter(1, 1, [&](int i) { fetchA(nxt, i); }, [&](int i) { copy(6 + i); });
    }
    // before the accumulators are read: the last quarter's results
    __device__ __forceinline__ void settle() {
#pragma unroll
        for (int s = 4; s < 8; ++s) mfma_settle(acc[s][4], acc[s][5], acc[s][6], acc[s][7]);
    }
};

}  // namespace gptq
