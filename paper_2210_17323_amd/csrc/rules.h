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

// ---- Hessian of [tokens, channels] activations: the tile of the kernel that reads them in place, 0: repacked ----
// For calls that the channel-major call makes without a workspace: one with a workspace repacks, to the same bytes as the token-major
// call does, and the two give the same bits.  That leaves fewer than 256 channels, up to 32768 tokens of fewer than 2048, and beyond, to 6144
// channels, ranges too short to be worth splitting (1889 tokens of 2048 to 3072 channels, 7073 of 4096, 15000 of 4608).
// Measured, us, in place with tiles of 128 (512 / tiles parts, at least one) / of 256 (the repacked kernel's parts) / repacked, float16:
//   2048 tokens: 1000 channels 19 / 29 / 42, 4096 77 / 86 / 108
//   4096:        4096 124 / 134 / 164, 6144 203 / 282 / 288
//   8192:        1536 39 / 49 / 69, 6144 368 / 485 / 451 (whole calls in place / repacked: 4608 226 / 272, 5120 271 / 285, 5632 292 / 298)
//   16384:       1664 68 / 79 / 96, 6144 708 / 901 / 750
//   32768:       1800 155 / 159 / 192
//   262144:      256 53 / 69 / 118
// Few channels always gain, tiles of 128 as long as they fill the chip in parts; in short calls the repack is most of the work
// whatever the channels; in between the larger tiles up to 4096 channels (8192 tokens of 2304 74 / 72 / 88, 3072 124 / 106 / 125).
constexpr int tokens_tile(int64_t n, int64_t t) {
    if (n <= 1920) return 128;
    if (n <= 4096) return t <= 6144 ? 128 : 256;
    return t <= 8192 ? 128 : 0;
}

// ---- float32 products with rows in whole tiles of 128 and K in whole steps: 128 x 128 tiles, or 256 rows (256 x 128 and larger) ----
// Small tiles where the larger ones leave CUs without any, for rows that are only whole tiles of 128, and where columns that end
// inside a tile make a second round of which at most half is filled: the small ones take half of such a round.  Measured at
// K = 1024, us, 256 x 128 / 128 x 128 / the guarded kernel: 4096 x 2050 (272 large tiles) 254 / 194 / 244, 8192 x 1026 (288) 254 / 193 / 245,
// 2048 x 6018 (384) 256 / 198 / 242, 4096 x 3202 (416) 258 / 257 / 328, 4096 x 4098 (528) 381 / 320 / 390.  Beyond two rounds a product alone still
// gains, but Alg. 1 on 12288 rows, whose strips run beside it, loses (10250 columns 12.5 ms against 13.0): the large tiles stay.
constexpr bool product_small_tiles(int64_t m, int64_t n) {
    const int64_t large = (m / 256) * ((n + 127) / 128);
    return m % 256 != 0 || large < 256 || (n % 128 != 0 && large <= 384);
}

// Triangular products (upper tiles of A B^T: float32 Hessians) with rows in whole tiles of 128 but not of 256, in short calls: what counts
// is how many workgroups start and end on a CU at a time, three of the guarded kernel's against two.  Measured, us, 128 x 128 direct-to-LDS
// tiles / guarded: 64 tokens of 1664 channels 10.4 / 10.7, 3968 19.8 / 20.1, 4224 26.5 / 25.0, 6272 43.5 / 41.3, 14464 227 / 206; 128 tokens of 4224 37.4 / 37.1, 5504 49.1 / 50.2,
// 6272 59.6 / 58.2, 14464 310 / 302; 192 tokens of 4224 48.2 / 49.0, 14464 405 / 404; 256 of 14464 492 / 508.
constexpr bool triangle_guarded(int64_t m, int64_t k) { return m % 256 != 0 && m > 4096 && k < (m > 6144 ? 192 : 128); }

// ---- Alg. 1: columns are walked in blocks of QB; one strip launch takes an outer block of up to QOB of them ----
constexpr int QB = 128;
constexpr int QOB = 1024;

// A group grid must see fully updated weights at its first column, so an outer block may only end where a group ends: groups
// that neither divide QOB nor are multiples of it fall back to outer blocks of one block.
constexpr int64_t alg1_outer_block(int64_t group) { return (group >= QB && (QOB % group) && (group % QOB)) ? QB : QOB; }

// Columns of block i that the strip launch over columns o0 .. o1 - 1 takes (0: none of them, QB or more: all).  It reads no
// working value past o1: a deferred update of those columns may still be running on the helper stream.
constexpr int64_t strip_block_columns(int64_t o0, int64_t o1, int i) { return o1 > o0 + (int64_t)i * QB ? o1 - (o0 + (int64_t)i * QB) : 0; }

// Rows that a CU takes at a time in a strip launch, 16 RT: it takes ceil(strips / CUs) rounds, and a strip through a whole outer block
// takes the microseconds below (mean of a first and a second outer block of 1024 columns, every CU with one strip; form 0 driven by
// U, 1 by R, 2 by R with groups inside a block; the walk alone is 80).  The walk is as long for 16 rows as for 48 -- one wavefront per
// 16 rows --, so few rows are spread thin over all CUs and many are taken 32 or 48 at a time.  Four row tiles do not fit in a CU's
// registers and LDS: they are two strips of two, one behind the other, 250 / 259 / 261 a round in long launches.  Calls on 2048 columns
// (two such launches and an update), us, four rounds of 48 rows / three of 64: 41216 rows 2326 / 2373, 2345 / 2433, 2524 / 2530; 45056 2365 / 2432,
// 2382 / 2471, 2564 / 2569; 49152 2432 / 2483, 2442 / 2538, 2618 / 2618.
constexpr int strip_row_tiles(int form, int64_t r) {
    constexpr int us[3][4] = {{94, 132, 182, 250}, {95, 136, 191, 259}, {98, 136, 194, 261}};
    int best = 1;
    int64_t best_us = 0;
    for (int rt = 1; rt <= 4; ++rt) {
        const int64_t strips = (r + 16 * rt - 1) / (16 * rt), t = (strips + 255) / 256 * us[form][rt - 1];
        if (rt == 1 || t < best_us) { best = rt; best_us = t; }
    }
    return best;
}

}  // namespace gptq
