// Ranges and rules of dispatch as plain functions, without HIP: the library and its CPU tests read the same ones.
#pragma once
#include <cstdint>

namespace gptq {

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
