// The serial part of step 2 (Section 3, Step 3): the 1024 x 1024 diagonal block of one outer block, R R^T with R upper triangular,
// taken from the last column backwards in blocks of 128, in ONE launch, and the inverses of its 128 x 128 diagonal blocks.
//
// Between workgroups.  Every 128 x 128 tile (i, k), i <= k, of the upper triangle has one workgroup that keeps it in accumulators:
//     C = H(i, k);  for c = last .. k + 1:  C -= P(i, c) P(k, c)^T;   then  P(i, k) = C R_kk^-T,  or R_kk from C where i = k
// What others need goes through memory with a counter each: stores and loads at agent scope, which pass the XCDs' own L2s, so
// nobody flushes a cache.  A diagonal tile hands out its panels of 16 columns as they are factored (L_p and the inverse of its
// 16 x 16 diagonal block), the tiles above it solve with them as they come, a tile's rows by one wavefront per 16 without a word to
// the others (a result is the next product's operand as it lies in the registers), and tile (k, k + 1) hands its columns on to
// diagonal tile k in the same way: when the last panel of R_k+1,k+1 is there, two products are left to do before R_kk is begun.
// Workgroups are numbered in the order in which their results are wanted and wait for lower numbers only.
//
// Inside a diagonal tile.  With rows and columns numbered from the last one, i' = 127 - i, this is the ordinary Cholesky
// factorisation L L^T, and R^-1 is L^-1; everything below is in that numbering.  Panels of 16 columns, p = 0 .. 7:
//   wavefronts 0, 1  A 16 x 16 diagonal block is factored by the 16 lanes of a DPP row, a row per lane, in registers: column j of
//           the block, needed by every lane, is register j, read from lane k of the own DPP row inside the multiply-add.
//           Every DPP row does this with its own copy of the block while its lanes solve another 16 rows of the panel with the
//           same broadcasts, so the panel below costs no more than the block.  The lanes whose rows are the diagonal block
//           itself solve the identity, which gives L_pp^-1.
//   wavefronts 2 .. 7  hold the rest of the matrix as 16 x 16 accumulators of v_mfma_f32_16x16x4_f32.  Behind a panel only the tiles of
//           the next one are updated before its pivots start; the others, and X = L^-1 -- X_pc = L_pp^-1 X_pc, then X_ic -=
//           L_ip X_pc for the rows below, a column of tiles per wavefront, so that a result is the next product's operand as it
//           lies in the registers --, are worked off beside the pivots.
// What bounds it is one chain, 23 us a block: 128 pivots with the tiles of the next panel between panels (15.4; 17.1 with 1 / sqrt(pivot) in
// the chain and two multiplications more a pivot), then the way of the last panel through tile (k, k + 1) to diagonal tile k: a counter is
// seen 0.5 us after it is raised, a load takes 0.8, a store 1.2.  An outer block takes 184 us.  As two launches per block, the
// factor of a diagonal tile and everything behind it in tiles of 64 x 64, it was 8 x (28 + 15) us and the gaps between them; as one launch
// in which a tile waits for the whole inverse of the diagonal block 240.
#include "chol_chain.h"

#include <utility>

namespace gptq {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

namespace {

constexpr int DB = 128, PB = 16, NP = DB / PB;
constexpr int PP = 20;                  // pitch of the panel in LDS (16-byte aligned rows on different banks)
constexpr int PW = DB + 4;              // pitch of a 128 x 128 operand in LDS
constexpr int OBW = 1024;
constexpr int WORKERS = 6;              // wavefronts 2 .. 7 of a diagonal tile
constexpr int CT = NP * (NP + 1) / 2 / WORKERS;                  // matrix tiles per worker: 6
constexpr int PAIR_FLAGS = NP * (NP - 1) / 2;
static_assert((PAIR_FLAGS + NP) * sizeof(int) <= CHAIN_FLAG_BYTES, "chol_chain.h states this size");

constexpr int tiles_before(int c) { return NP * c - c * (c - 1) / 2; }        // of the columns left of column c
// tile number -> (i, c), i >= c, of the lower triangle with its diagonal, column by column
__device__ __forceinline__ void tile_of(int t, int& i, int& c) { c = 0; while (t >= NP - c) { t -= NP - c; ++c; } i = c + t; }

// w -= m * (u of lane C of the own DPP row)
template <int C>
__device__ __forceinline__ void fma_bcast16(float& w, float u, float m) {
    asm volatile("v_fmac_f32_dpp %0, %1, -%2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(w) : "v"(u), "v"(m), "n"(C));
}
template <int C>
__device__ __forceinline__ float bcast16(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x150 + C, 0xf, 0xf, true));     // row_newbcast
}
// v is made here: between the statements before and after, not where the compiler would rather have it
__device__ __forceinline__ void here(float& v) { asm volatile("" : "+v"(v)); }

template <int J, int FIRST, int LAST>
__device__ __forceinline__ void update_right(float (&dx)[PB], float (&px)[PB], float du, float pu) {
    if constexpr (FIRST < LAST && FIRST < PB) {
        fma_bcast16<FIRST>(dx[FIRST], dx[J], du);
        fma_bcast16<FIRST>(px[FIRST], dx[J], pu);
        update_right<J, FIRST + 1, LAST>(dx, px, du, pu);
    }
}

// Pivot J, whose reciprocal is in r: the columns right of it lose their products with column J, which stays as it is until all
// pivots are known -- an element loses column * (row / pivot), one product with one rounding before it.  Column J + 1 is
// first, and the reciprocal of its pivot -- the hardware's estimate with one Newton step -- is made between the other columns.
// `mine` keeps the pivot of this lane's row.
template <int J>
__device__ __forceinline__ void pivot(float (&dx)[PB], float (&px)[PB], float dd, float r, float& mine, int l16) {
    mine = l16 == J ? dd : mine;
    if constexpr (J + 1 < PB) {
        const float du = dx[J] * r, pu = px[J] * r;
        update_right<J, J + 1, J + 3>(dx, px, du, pu);
        if constexpr (J + 2 < PB) here(dx[J + 1]); else asm volatile("s_nop 1" : "+v"(dx[J + 1]));      // two wait states between a vector write and a DPP read of it
        float dn = bcast16<J + 1>(dx[J + 1]);
        float est = __builtin_amdgcn_rcpf(dn);
        here(est);
        update_right<J, J + 3, J + 5>(dx, px, du, pu);
        float e = fmaf(-dn, est, 1.f);
        here(e);
        update_right<J, J + 5, J + 6>(dx, px, du, pu);
        float rn = fmaf(e, est, est);
        here(rn);
        update_right<J, J + 6, PB>(dx, px, du, pu);
        pivot<J + 1>(dx, px, dn, rn, mine, l16);
    }
}

template <int... J>
__device__ __forceinline__ void scale_columns(float (&x)[PB], float inv, std::integer_sequence<int, J...>) { ((x[J] *= bcast16<J>(inv)), ...); }

__device__ __forceinline__ void barrier_lds() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
// ... and every global store of the workgroup has reached the memory the other XCDs see
__device__ __forceinline__ void barrier_all() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Loads and stores that other workgroups' stores and loads of the same launch meet: agent scope, past the XCD's own caches.
__device__ __forceinline__ floatx4 load_shared(const float* p) {
    const uint64_t* q = reinterpret_cast<const uint64_t*>(p);
    const uint64_t a = __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), b = __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return floatx4{__uint_as_float((uint32_t)a), __uint_as_float((uint32_t)(a >> 32)), __uint_as_float((uint32_t)b), __uint_as_float((uint32_t)(b >> 32))};
}
__device__ __forceinline__ void store_shared(float* p, floatx4 v) {
    uint64_t* q = reinterpret_cast<uint64_t*>(p);
    __hip_atomic_store(q, (uint64_t)__float_as_uint(v[0]) | ((uint64_t)__float_as_uint(v[1]) << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(q + 1, (uint64_t)__float_as_uint(v[2]) | ((uint64_t)__float_as_uint(v[3]) << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_shared(float* p, float v) {
    __hip_atomic_store(reinterpret_cast<uint32_t*>(p), __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct ChainArgs { float* H; int64_t ld; int64_t o0; int ow; float* dinv; float* panel; float* packed; int* flags; int epoch; int* info; };

// Counters: columns of P(i, k) and panels of R_kk that are in memory, in sixteens, on top of 16 times the epoch.
__device__ __forceinline__ int pair_flag(int i, int k) { return k * (k - 1) / 2 + i; }
__device__ __forceinline__ int diag_flag(int k) { return PAIR_FLAGS + k; }

// A wait ends when the counter is there.  It ends after WAIT_TICKS of the 100 MHz clock too, with CHAIN_TIMED_OUT in *info, so that a
// workgroup whose partner never starts leaves all the same; nothing more is waited for then.  The clock runs on while the process is
// scheduled off, so what passes between two reads of the counter counts as POLL_TICKS at most, and the last thing before giving up is a read.
constexpr uint64_t WAIT_TICKS = 1000000000ull;           // 10 s
constexpr uint64_t POLL_TICKS = 100000ull;               // 1 ms
struct Counters {
    const ChainArgs& g;
    int base;
    bool lost = false;
    __device__ explicit Counters(const ChainArgs& a) : g(a), base(16 * a.epoch) {}
    __device__ __forceinline__ int read(int f) const { return __hip_atomic_load(g.flags + f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - base; }
    // by one thread: the count, once it is at least `want`
    __device__ __forceinline__ int wait(int f, int want) {
        int v = read(f);
        if (v >= want) return v;
        if (lost) return NP;
        uint64_t waited = 0, last = __builtin_amdgcn_s_memrealtime();
        do {
            __builtin_amdgcn_s_sleep(1);
            const uint64_t now = __builtin_amdgcn_s_memrealtime();
            waited += min(now - last, POLL_TICKS);
            last = now;
            v = read(f);
            if (v >= want) return v;
        } while (waited <= WAIT_TICKS);
        lost = true;
        atomicCAS(g.info, 0, CHAIN_TIMED_OUT);
        return NP;
    }
    __device__ __forceinline__ void raise(int f, int count) const { __hip_atomic_store(g.flags + f, base + count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
};

// The panels of 16 columns of somebody else's tile, 128 rows each, into LDS (pitch PP), all that are there at a time.
struct PanelStream {
    Counters& c;
    int flag;
    const float* src;                   // this thread's four columns of its row, of panel 0
    int step;                           // from there to the next panel's
    float* lds;                         // NP panels
    int* slot;                          // a word of LDS
    int loaded = 0;
    // Panel p, for everybody.  When panels came, `came` is called: every store that the workgroup made before this call is in memory.
    template <int p, class F>
    __device__ __forceinline__ const float* get(F came) {
        if (loaded <= p) {
            if (threadIdx.x == 0) *slot = c.wait(flag, p + 1);
            barrier_lds();
            loaded = __builtin_amdgcn_readfirstlane(*slot);
            floatx4 v[NP];
#pragma unroll
            for (int q = p; q < NP; ++q) if (q < loaded) v[q] = load_shared(src + q * step);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
            for (int q = p; q < NP; ++q)
                if (q < loaded) *reinterpret_cast<floatx4*>(&lds[q * (DB * PP) + (threadIdx.x >> 2) * PP + (threadIdx.x & 3) * 4]) = v[q];
            barrier_lds();
            came();
        }
        return lds + p * (DB * PP);
    }
};

// P(i, c) into LDS, [row][k]
__device__ __forceinline__ void request_panel(const ChainArgs& g, int i, int c, floatx4 (&v)[8]) {
    const float* p = g.panel + (int64_t)(DB * i + (threadIdx.x >> 5)) * OBW + DB * c + (threadIdx.x & 31) * 4;
#pragma unroll
    for (int t = 0; t < 8; ++t) v[t] = load_shared(p + 16 * t * OBW);
}
__device__ __forceinline__ void put_panel(float* lds, const floatx4 (&v)[8]) {
#pragma unroll
    for (int t = 0; t < 8; ++t) *reinterpret_cast<floatx4*>(&lds[((threadIdx.x >> 5) + 16 * t) * PW + (threadIdx.x & 31) * 4]) = v[t];
}

}  // namespace

__global__ __launch_bounds__(512) void chol_chain_kernel(ChainArgs g) {
    __shared__ __attribute__((aligned(16))) float pa[2 * DB * PW];
    __shared__ int slot;
    float* const pb = pa + DB * PW;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, kq = lane >> 4;
    const int nb = (g.ow + DB - 1) / DB;
    // Panels whose products are subtracted at once, not summed with those of the later ones: up to the first one of the outer block that is not past
    // its end.  Where the channels have much in common (inputs behind a ReLU) its first column carries that, and a sum that
    // began with it would be rounded at its size ever after, not at the size of what it leaves.  The column comes in the last of the panel's products.
    auto first_panel = [&](int q) { return q == nb - 1 ? (DB - min(DB, g.ow - DB * q)) / PB : -1; };
    // workgroup -> tiles: column by column from the last, the diagonal tile first, then upwards
    int k = nb - 1, m = (int)blockIdx.x;
    while (m > k) { m -= k + 1; --k; }
    Counters counters(g);
    // the packed outer block, as the strips of rows above it read it: [wavefront: 32 columns][16 k][even, odd columns][lane][4 k], the
    // inverses of the diagonal blocks from the last on, then the tiles above them (chol_strip.h)
    auto packed_word = [](int n, int kk) { return ((((n >> 5) * 8 + (kk >> 4)) * 2 + (n & 1)) * 64 + ((n >> 1) & 15) + 16 * ((kk >> 2) & 3)) * 4 + (kk & 3); };

    if (m > 0) {
        // ---- tile (i, k): wavefront w holds rows 16 w .. 16 w + 15, transposed -- lane l16 is the row, element e of tile j the (reversed)
        //      column 16 j + 4 kq + e
        const int i = k - m;
        const int width = min(DB, g.ow - DB * k);        // columns that exist; rows all do
        const int row = 16 * wave + l16;
        auto col = [&](int j) { return DB - 4 - 16 * j - 4 * kq; };              // of the first of the four columns of tile j, ascending
        float* hrow = g.H + (g.o0 + DB * i + row) * g.ld + g.o0 + DB * k;
        float* prow = g.panel + (int64_t)(DB * i + row) * OBW + DB * k;
        floatx4 C[NP];
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const int c = col(j);
            if (c + 4 <= width) {
                const floatx4 h = *reinterpret_cast<const floatx4*>(hrow + c);
                C[j] = floatx4{h[3], h[2], h[1], h[0]};
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) C[j][e] = c + 3 - e < width ? hrow[c + 3 - e] : 0.f;
            }
        }
#pragma unroll 1
        for (int c = nb - 1; c > k; --c) {
            if (tid == 0) { counters.wait(pair_flag(i, c), NP); counters.wait(pair_flag(k, c), NP); }
            barrier_lds();                               // both are there, and nobody reads the operands of the round before
            {
                floatx4 va[8], vb[8];
                request_panel(g, i, c, va);
                request_panel(g, k, c, vb);
                put_panel(pa, va);
                put_panel(pb, vb);
            }
            barrier_lds();
            floatx4 acc[NP];
#pragma unroll
            for (int j = 0; j < NP; ++j) acc[j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
            for (int t = 0; t < 8; ++t) {
                const floatx4 b = *reinterpret_cast<const floatx4*>(&pa[row * PW + 16 * t + 4 * kq]);
                floatx4 a[NP];
#pragma unroll
                for (int j = 0; j < NP; ++j) a[j] = *reinterpret_cast<const floatx4*>(&pb[(DB - 1 - 16 * j - l16) * PW + 16 * t + 4 * kq]);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int j = 0; j < NP; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j][e], b[e], acc[j], 0, 0, 0);
            }
            // a panel's 128 products are summed on their own and subtracted once: one by one, each would be rounded at C's size
#pragma unroll
            for (int j = 0; j < NP; ++j) C[j] -= acc[j];
        }
        barrier_lds();
        // P = C R_kk^-T, column block by column block: P_p^T = L_pp^-1 (C_p^T - sum), then L_jp P_p^T onto the sums of the later ones.
        // (What the first panels leave goes to C at once, first_panel.)
        const int first = first_panel(k);
        PanelStream L{counters, diag_flag(k), g.panel + (int64_t)(DB * k + (tid >> 2)) * OBW + DB * k + (tid & 3) * 4, PB, pa, &slot};
        floatx4 S[NP];
#pragma unroll
        for (int j = 0; j < NP; ++j) S[j] = floatx4{0.f, 0.f, 0.f, 0.f};
        auto solve = [&](auto P) {
            constexpr int p = decltype(P)::value;
            const float* lp = L.template get<p>([&] {
                // diagonal tile i takes its neighbour's columns as they come; nobody else wants less than all of them
                if (p > 0 && m == 1 && tid == 0) counters.raise(pair_flag(i, k), p);
            });
            floatx4 cur = {0.f, 0.f, 0.f, 0.f};
            const floatx4 rhs = C[p] - S[p];
#pragma unroll
            for (int e = 0; e < 4; ++e) cur = __builtin_amdgcn_mfma_f32_16x16x4f32(lp[(PB * p + 4 * kq + e) * PP + l16], rhs[e], cur, 0, 0, 0);
            C[p] = cur;
            store_shared(prow + col(p), floatx4{cur[3], cur[2], cur[1], cur[0]});
#pragma unroll
            for (int j = p + 1; j < NP; ++j) {
                const floatx4 a = *reinterpret_cast<const floatx4*>(&lp[(PB * j + l16) * PP + 4 * kq]);
#pragma unroll
                for (int e = 3; e >= 0; --e) S[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], cur[e], S[j], 0, 0, 0);
            }
            if (p <= first) {
#pragma unroll
                for (int j = p + 1; j < NP; ++j) { C[j] -= S[j]; S[j] = floatx4{0.f, 0.f, 0.f, 0.f}; }
            }
        };
        [&]<int... P>(std::integer_sequence<int, P...>) { (solve(std::integral_constant<int, P>{}), ...); }(std::make_integer_sequence<int, NP>{});
        barrier_all();
        if (tid == 0) counters.raise(pair_flag(i, k), NP);
        const int s = nb - 1 - k, s2 = nb - 1 - i;       // positions in the order of the walk
        float* packed = g.packed ? g.packed + (int64_t)(NP + s * (2 * NP - 1 - s) / 2 + s2 - s - 1) * (DB * DB) : nullptr;
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const int c = col(j);
            const floatx4 v = {C[j][3], C[j][2], C[j][1], C[j][0]};
            if (c + 4 <= width) *reinterpret_cast<floatx4*>(hrow + c) = v;
            else {
#pragma unroll
                for (int e = 0; e < 4; ++e) if (c + e < width) hrow[c + e] = v[e];
            }
            if (packed) *reinterpret_cast<floatx4*>(packed + packed_word(row, c)) = v;
        }
        return;
    }

    // ---- the diagonal tile: wavefronts 2 .. 7, six 16 x 16 tiles each
    const int worker = wave - 2;
    floatx4 ch[CT];
    int ci[CT], cc[CT];
    const int nbk = min(DB, g.ow - DB * k);
    float* Hblk = g.H + (g.o0 + DB * k) * g.ld + g.o0 + DB * k;
    if (worker >= 0) {
#pragma unroll
        for (int s = 0; s < CT; ++s) {
            tile_of(worker + WORKERS * s, ci[s], cc[s]);
#pragma unroll
            for (int e = 0; e < 4; ++e) {                // element (16 i + 4 kq + e, 16 c + l16) of the reversed block
                const int a = DB - 1 - (PB * ci[s] + 4 * kq + e), b = DB - 1 - (PB * cc[s] + l16);
                ch[s][e] = (a < nbk && b < nbk) ? Hblk[(int64_t)min(a, nbk - 1) * g.ld + min(b, nbk - 1)] : (a == b ? 1.f : 0.f);
            }
        }
    }
    float* dinv = g.dinv + (int64_t)k * (DB * DB);
    float* packed = g.packed ? g.packed + (int64_t)(nb - 1 - k) * (DB * DB) : nullptr;
    for (int q = tid; q < DB * DB / 4; q += 512) {       // R^-1 below its diagonal
        const int row = q >> 5, c = (q & 31) * 4;
        if ((c | 15) >= row) continue;
        *reinterpret_cast<floatx4*>(dinv + row * DB + c) = floatx4{0.f, 0.f, 0.f, 0.f};
        if (packed) *reinterpret_cast<floatx4*>(packed + packed_word(row, c)) = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    // ch -= P P^T, P in LDS
    auto update_diagonal = [&](const float* p) {
#pragma unroll
        for (int s = 0; s < CT; ++s) {
            const float* arow = &p[(DB - 1 - (PB * ci[s] + l16)) * PW + 4 * kq];
            const float* brow = &p[(DB - 1 - (PB * cc[s] + l16)) * PW + 4 * kq];
            floatx4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const floatx4 a = *reinterpret_cast<const floatx4*>(arow + 16 * t), b = *reinterpret_cast<const floatx4*>(brow + 16 * t);
#pragma unroll
                for (int e = 0; e < 4; ++e) v = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], v, 0, 0, 0);
            }
            ch[s] -= v;
        }
    };

#pragma unroll 1
    for (int c = nb - 1; c > k + 1; --c) {
        if (tid == 0) counters.wait(pair_flag(k, c), NP);
        barrier_lds();
        {
            floatx4 v[8];
            request_panel(g, k, c, v);
            put_panel(pa, v);
        }
        barrier_lds();
        if (worker >= 0) update_diagonal(pa);
    }

    // ---- the diagonal tile is factored
    float* const own = pa + NP * (DB * PP);              // behind the panels of the tile to the right
    auto panel = [&](int p) { return own + (p & 1) * (DB * PP); };              // columns 16 p .. of rows 16 p ..: before, then L
    auto linv = [&](int p) { return own + 2 * (DB * PP) + (p & 1) * (PB * PP); };               // L_pp^-1, column by column
    auto lpp = [&](int p) { return own + 2 * (DB * PP) + (2 + (p & 1)) * (PB * PP); };          // L_pp
    auto big_flag = [&](int p) { return reinterpret_cast<int*>(own + 2 * (DB * PP) + 4 * PB * PP) + p; };          // the diagonal of block p reaches 2^100
    int bad_col = -1;
    // columns of X: worker v has column v, worker 4 also column 7 and worker 5 column 6, of which only tile (7, 6) waits
    floatx4 xa[NP], xb = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < NP; ++i) xa[i] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int cb = worker == 4 ? 7 : (worker == 5 ? 6 : NP);
    auto store_dinv = [&](int i, int c, floatx4 v) {     // X_ic is R^-1 at rows 127 - 16 i - .., columns 127 - 16 c - ..
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = DB - 1 - (PB * i + 4 * kq + e), col = DB - 1 - (PB * c + l16);
            dinv[row * DB + col] = v[e];
            if (packed) packed[packed_word(row, col)] = v[e];
        }
    };
    auto update_tile = [&](floatx4& d, const float* pn, int i, int c) {
        const floatx4 a = *reinterpret_cast<const floatx4*>(&pn[(PB * i + l16) * PP + 4 * kq]);
        const floatx4 b = *reinterpret_cast<const floatx4*>(&pn[(PB * c + l16) * PP + 4 * kq]);
        floatx4 v = {0.f, 0.f, 0.f, 0.f};                // the panel's 16 products, subtracted at once: one by one, each would
#pragma unroll
        for (int e = 0; e < 4; ++e) v = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], v, 0, 0, 0);      // be rounded at the size of the element
        d -= v;
    };
    auto extract = [&](floatx4 v, int i, int p) {        // tile (i, p)
        float* pn = panel(p);
#pragma unroll
        for (int e = 0; e < 4; ++e) pn[(PB * i + 4 * kq + e) * PP + l16] = v[e];
        if (i == p) {
            bool big = false;
#pragma unroll
            for (int e = 0; e < 4; ++e) big |= 4 * kq + e == l16 && v[e] >= 0x1p100f;
            const bool any = __ballot(big) != 0;
            if (lane == 0) *big_flag(p) = any;
        }
    };
    // what panel p leaves to do beside the next one's pivots
    auto behind = [&](auto P) {
        constexpr int p = decltype(P)::value;
        const float* pn = panel(p);
        const float* li = linv(p);
        // to the tiles above: rows 16 p .. of the panel, the inverse of its diagonal block in the place of the block
        if (k > 0)
        for (int q = tid - 128; q < (DB - PB * p) * 4; q += 64 * WORKERS) {
            const int row = PB * p + (q >> 2), c = (q & 3) * 4;
            const floatx4 v = row < PB * (p + 1) ? *reinterpret_cast<const floatx4*>(&li[(row - PB * p) * PP + c]) : *reinterpret_cast<const floatx4*>(&pn[row * PP + c]);
            store_shared(g.panel + (int64_t)(DB * k + row) * OBW + DB * k + PB * p + c, v);
        }
        if (p + 1 == NP && worker == 0) {                // the last panel is this wavefront's alone, and somebody waits for it
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (lane == 0) counters.raise(diag_flag(k), NP);
        }
#pragma unroll
        for (int s = 0; s < CT; ++s)
            if (WORKERS * s >= tiles_before(p + 2) || (WORKERS * s + WORKERS - 1 >= tiles_before(p + 2) && cc[s] > p + 1)) update_tile(ch[s], pn, ci[s], cc[s]);
        const floatx4 lx = *reinterpret_cast<const floatx4*>(&li[l16 * PP + 4 * kq]);      // X_pp, as it lies in accumulators
        floatx4 la;                                      // ... and as the first operand
#pragma unroll
        for (int e = 0; e < 4; ++e) la[e] = li[(4 * kq + e) * PP + l16];
        auto scaled = [&](floatx4 old) {
            floatx4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int e = 0; e < 4; ++e) v = __builtin_amdgcn_mfma_f32_16x16x4f32(la[e], old[e], v, 0, 0, 0);
            return v;
        };
        auto below = [&](floatx4& x, floatx4 cur, int i) {
            const floatx4 a = *reinterpret_cast<const floatx4*>(&pn[(PB * i + l16) * PP + 4 * kq]);
            floatx4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int e = 0; e < 4; ++e) v = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], cur[e], v, 0, 0, 0);
            x -= v;
        };
        if (worker <= p) {
            floatx4 cur = lx;
            if (worker < p) cur = scaled(xa[p]);
            store_dinv(p, worker, cur);
#pragma unroll
            for (int i = p + 1; i < NP; ++i) below(xa[i], cur, i);
        }
        if (cb <= p) {
            floatx4 cur = lx;
            if (cb < p) cur = scaled(xb);              // only column 6 at panel 7
            store_dinv(p, cb, cur);
            if (p == 6) below(xb, cur, 7);
        }
        // R: rows 127 - 16 p and up, columns 127 - 16 p - 15 .. 127 - 16 p
        const int b0 = DB - 1 - PB * p - 15;
        for (int q = tid - 128; q < (DB - PB * p) * 4; q += 64 * WORKERS) {
            const int row = PB * p + (q >> 2), c = (q & 3) * 4, a = DB - 1 - row;
            const floatx4 v = row < PB * (p + 1) ? *reinterpret_cast<const floatx4*>(&lpp(p)[(row - PB * p) * PP + 12 - c])
                                                 : *reinterpret_cast<const floatx4*>(&pn[row * PP + 12 - c]);
            if (a >= nbk) continue;
            float* dst = Hblk + (int64_t)a * g.ld + b0 + c;
            if (b0 + c + 4 <= nbk) *reinterpret_cast<floatx4*>(dst) = floatx4{v[3], v[2], v[1], v[0]};
            else {
#pragma unroll
                for (int e = 0; e < 4; ++e) if (b0 + c + e < nbk) dst[e] = v[3 - e];
            }
        }
    };
    barrier_lds();                                       // nobody reads the last of the panels above any more
    // the columns of P(k, k + 1) as they come; behind the last two only the tiles of the first panel are updated before the
    // pivots start
    floatx4 sum[CT];
#pragma unroll
    for (int s = 0; s < CT; ++s) sum[s] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto add_tile = [&](int s, const float* pp) {
        const floatx4 a = *reinterpret_cast<const floatx4*>(&pp[(DB - 1 - (PB * ci[s] + l16)) * PP + 4 * kq]);
        const floatx4 b = *reinterpret_cast<const floatx4*>(&pp[(DB - 1 - (PB * cc[s] + l16)) * PP + 4 * kq]);
#pragma unroll
        for (int e = 3; e >= 0; --e) sum[s] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], sum[s], 0, 0, 0);
    };
    if (k + 1 < nb) {
        const int first = first_panel(k + 1);
        PanelStream S{counters, pair_flag(k, k + 1), g.panel + (int64_t)(DB * k + (tid >> 2)) * OBW + DB * (k + 1) + DB - PB + (tid & 3) * 4, -PB, pa, &slot};
        auto take = [&](auto P) {
            constexpr int p = decltype(P)::value;
            const float* pp = S.template get<p>([] {});
            if (worker >= 0) {
#pragma unroll
                for (int s = 0; s < CT; ++s)
                    if (p + 2 < NP || (WORKERS * s < tiles_before(1) && cc[s] == 0)) add_tile(s, pp);
                if (p <= first) {
#pragma unroll
                    for (int s = 0; s < CT; ++s) { ch[s] -= sum[s]; sum[s] = floatx4{0.f, 0.f, 0.f, 0.f}; }
                }
            }
        };
        [&]<int... P>(std::integer_sequence<int, P...>) { (take(std::integral_constant<int, P>{}), ...); }(std::make_integer_sequence<int, NP>{});
    }
    if (worker >= 0) {
#pragma unroll
        for (int s = 0; s < CT; ++s)
            if (WORKERS * s < tiles_before(1) && cc[s] == 0) {
                ch[s] -= sum[s];
                extract(ch[s], ci[s], 0);
            }
    }
    barrier_lds();
    if (wave < 2) {
#pragma unroll 1
        for (int p = 0; p < NP; ++p) {
            float* pn = panel(p);
            if (64 * wave + 63 >= PB * p) {
                const int row = 64 * wave + lane;        // the row of the panel this lane solves
                const bool own = (row >> 4) == p;        // ... the diagonal block's: the identity instead
                float dx[PB], px[PB];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const floatx4 d = *reinterpret_cast<const floatx4*>(&pn[(PB * p + l16) * PP + 4 * q]);
                    const floatx4 x = *reinterpret_cast<const floatx4*>(&pn[max(row, PB * p) * PP + 4 * q]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        dx[4 * q + e] = d[e];
                        px[4 * q + e] = own ? (l16 == 4 * q + e ? 1.f : 0.f) : x[e];
                    }
                }
                // A pivot's reciprocal must not be denormal: a block whose diagonal (no pivot is larger) comes near the end of the
                // float range is factored as 2^-64 of it, exactly.
                const bool big = *big_flag(p) != 0;
                if (big) {
#pragma unroll
                    for (int q = 0; q < PB; ++q) { dx[q] *= 0x1p-64f; px[q] *= 0x1p-64f; }
                }
                float mine = 0.f;
                {
                    const float dd = bcast16<0>(dx[0]);
                    const float est = __builtin_amdgcn_rcpf(dd);
                    pivot<0>(dx, px, dd, fmaf(fmaf(-dd, est, 1.f), est, est), mine, l16);
                }
                asm volatile("s_nop 1" ::: "memory");
                // 1 / sqrt(pivot) of the lane's own pivot: the estimate with one Newton step whose residual 1 - pivot * inv^2 is taken
                // without the rounding of pivot * inv (half an ulp in all: the first digit the whole factorisation loses)
                const float est = __builtin_amdgcn_rsqf(mine);
                const float t = mine * est;
                float inv = fmaf(0.5f * est, fmaf(-fmaf(mine, est, -t), est, fmaf(-t, est, 1.f)), est);
                if (big) inv *= 0x1p32f;
                scale_columns(px, inv, std::make_integer_sequence<int, PB>{});
                if (own) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) *reinterpret_cast<floatx4*>(&linv(p)[l16 * PP + 4 * q]) = floatx4{px[4 * q], px[4 * q + 1], px[4 * q + 2], px[4 * q + 3]};
                } else if (row > PB * p) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) *reinterpret_cast<floatx4*>(&pn[row * PP + 4 * q]) = floatx4{px[4 * q], px[4 * q + 1], px[4 * q + 2], px[4 * q + 3]};
                }
                const uint32_t bad = (uint32_t)__ballot(!(mine > 0.f)) & 0xffffu;
                if (bad && bad_col < 0) bad_col = PB * p + __builtin_ctz(bad);
                if (own) {
                    const float root = __fsqrt_rn(mine) * (big ? 0x1p32f : 1.f);              // the diagonal of L
                    scale_columns(dx, inv, std::make_integer_sequence<int, PB>{});
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        floatx4 v;
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] = 4 * q + e < l16 ? dx[4 * q + e] : (4 * q + e == l16 ? root : 0.f);
                        *reinterpret_cast<floatx4*>(&lpp(p)[l16 * PP + 4 * q]) = v;
                    }
                }
            }
            barrier_lds();
            barrier_lds();
        }
    } else {
        auto step = [&](auto P) {
            constexpr int p = decltype(P)::value;
            if constexpr (p > 0) {
                behind(std::integral_constant<int, p - 1>{});
            } else {
#pragma unroll
                for (int s = 0; s < CT; ++s)
                    if (WORKERS * s + WORKERS - 1 >= tiles_before(1) && cc[s] > 0) {
                        if (k + 1 < nb) { add_tile(s, pa + (NP - 2) * (DB * PP)); add_tile(s, pa + (NP - 1) * (DB * PP)); }
                        ch[s] -= sum[s];
                    }
            }
            barrier_lds();
            if constexpr (p + 1 < NP) {
#pragma unroll
                for (int s = 0; s < CT; ++s)
                    if (WORKERS * s + WORKERS - 1 >= tiles_before(p + 1) && WORKERS * s < tiles_before(p + 2) && cc[s] == p + 1) {
                        update_tile(ch[s], panel(p), ci[s], cc[s]);
                        extract(ch[s], ci[s], p + 1);
                    }
            }
            barrier_all();
            if constexpr (p > 0) { if (tid == 128) counters.raise(diag_flag(k), p); }
        };
        [&]<int... P>(std::integer_sequence<int, P...>) { (step(std::integral_constant<int, P>{}), ...); }(std::make_integer_sequence<int, NP>{});
        behind(std::integral_constant<int, NP - 1>{});
    }
    if (bad_col >= 0 && lane == 0) atomicCAS(g.info, 0, (int)g.o0 + DB * k + DB - bad_col);     // column 127 - bad_col, counted from 1
}

int launch_chol_chain(float* H, int64_t ld, int64_t o0, int ow, float* dinv, float* panel, float* packed, int* flags, int epoch, int* info, hipStream_t s) {
    const ChainArgs g{H, ld, o0, ow, dinv, panel, packed, flags, epoch, info};
    const int nb = (ow + DB - 1) / DB;
    hipLaunchKernelGGL(chol_chain_kernel, dim3((unsigned)(nb * (nb + 1) / 2)), dim3(512), 0, s, g);
    GPTQ_LAUNCH_CHECK();
    return GPTQ_OK;
}

}  // namespace gptq
