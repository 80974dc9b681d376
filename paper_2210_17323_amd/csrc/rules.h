// Ranges and rules of dispatch as plain functions, without HIP: the library and its CPU tests read the same ones.
#pragma once
#include <cstdint>

namespace gptq {

// ---- Hessian of float32 activations (channel-major): the kernel of small tiles or the float32 product ----
// Both take rounds of one tile per CU, n (n + 1) / 2 over 64 x 64 or 128 x 128 of them.  Measured for 4096 tokens: 118 us a round of
// small tiles (n = 1408: 135 us, 1984: 247, 2056: 349, 2500: 455, 2900: 565); the product 250 us a round where rows and tokens
// come in whole tiles (n = 1536: 250, 2560: 255, 3072: 486), and through its guarded kernel 385 for up to 256 tiles (n = 1544: 372, 2500: 388),
// 630 for up to 325 (n = 2824: 614, 3072: 650).  One round of small tiles is always the faster, two are from where the guarded kernel or
// a long call would be the other choice (n = 1664, 64 tokens: 14 us against 12, 512: 43 against 38, 4096: 247 against 251); beyond, only
// where the product would be guarded and the call is long enough for rounds to be what it takes (512 tokens of 2056 channels: 59 us
// against 57, 2700: 81 against 63, 2950: 100 against 91).
constexpr int64_t hessian_rounds(int64_t n, int64_t tile) { return (((n + tile - 1) / tile) * ((n + tile - 1) / tile + 1) / 2 + 255) / 256; }
constexpr bool hessian_f32_small_tiles(int64_t n, int64_t t) {
    if (n > 3072) return false;
    const int64_t rounds = hessian_rounds(n, 64);
    const bool whole = n % 128 == 0 && t % 64 == 0;
    if (rounds == 1) return true;
    if (t < 1024) return rounds == 2 && !whole;
    if (rounds == 2) return true;
    return !whole && 118 * rounds < (hessian_rounds(n, 128) == 1 ? 385 : 630);
}

// ---- Alg. 1: columns are walked in blocks of QB; one strip launch takes an outer block of up to QOB of them ----
constexpr int QB = 128;
constexpr int QOB = 1024;

// A group grid must see fully updated weights at its first column, so an outer block may only end where a group ends: groups
// that neither divide QOB nor are multiples of it fall back to outer blocks of one block.
constexpr int64_t alg1_outer_block(int64_t group) { return (group >= QB && (QOB % group) && (group % QOB)) ? QB : QOB; }

// Columns of block i that the strip launch over columns o0 .. o1 - 1 takes (0: none of them, QB or more: all).  It reads no
// working value past o1: a deferred update of those columns may still be running on the helper stream.
constexpr int64_t strip_block_columns(int64_t o0, int64_t o1, int i) { return o1 > o0 + (int64_t)i * QB ? o1 - (o0 + (int64_t)i * QB) : 0; }

}  // namespace gptq
