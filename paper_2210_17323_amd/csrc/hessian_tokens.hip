// Step 1 for activations as a layer has them, X [tokens, channels], read in place: H += 2 X^T X.
//
// A matrix operand wants consecutive tokens of one channel in a lane; X has consecutive channels.  The panels go into LDS as they
// lie -- 32 tokens x 128 or 256 channels, whole lines of memory -- and are turned on the way out of it: ds_read_b64_tr_b16 hands 16 lanes
// a 4 x 16 block transposed, four tokens of one channel each.  A token's row starts on bank 0 (256 or 512 bytes), so its 16-byte
// chunks are swizzled by the token: the four rows a transposed read takes lie on different banks.
// Otherwise the pipeline of the repacked kernel: five LDS stages filled by global_load_lds, one bare barrier per step, the next
// step's first operands read across it.  Tokens past the last one are read from a block of zeros.
// A tile of 128 x 128 (4 wavefronts of 64 x 64) is bound by LDS, one of 256 x 256 (128 x 128 each) by the matrix cores; few tiles get their
// token range split into parts, whose partial tiles are added in the order of their ranges (the same bits from every call).
// Against a repack and the repacked kernel, a call of float16 tokens, us: 256 channels x 16384 tokens 38 -> 23, 1000 x 16400 64 -> 37, 1536 x 32768 138 ->
// 105, 2000 x 32000 196 -> 159, 2048 x 1880 75 -> 27, 4096 x 2048 107 -> 77, 4096 x 6500 220 -> 184, 5632 x 8192 298 -> 292, 6144 x 2048 191 -> 121.
// Where the repack is little beside the products the repacked kernel's 16-byte reads win (6144 channels x 16384: 750 against 708 and 901);
// tokens_tile in rules.h has the line, and which calls may come here.
#include "hessian_tokens.h"
#include "syrk_tiles.h"

namespace gptq {

typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

namespace {

constexpr int STEP = 32, TRIP = 5;      // tokens per step, steps per trip of the loop

__device__ const uint4 token_zeros[1] = {{0u, 0u, 0u, 0u}};

struct TokenArgs {
    float* H; int64_t ldh; const uint16_t* X; int64_t ldx, n, t;
    int nt; int64_t total;              // tiles per side, tiles
    int parts; int64_t trips;           // parts of the token range, trips in all
    float* P;                           // partial tiles [tile][part][tile x tile], or null
};

template <bool BF16, int WT>            // WT: 32-channel MFMA tiles per side of a wavefront's tile
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WT == 4 ? 1 : 2, WT == 4 ? 1 : 2))) void syrk_tokens_kernel(TokenArgs g) {
    constexpr int TILE = 64 * WT, ROW = TILE * 2, PANEL = STEP * ROW, COPIES = PANEL / 4096;      // bytes of a token's row and of a panel; copies per wavefront and panel
    constexpr int RPC = 1024 / ROW;                          // token rows per copy
    __shared__ __attribute__((aligned(16))) unsigned char stage0[2 * PANEL];
    __shared__ __attribute__((aligned(16))) unsigned char stage1[2 * PANEL];
    __shared__ __attribute__((aligned(16))) unsigned char stage2[2 * PANEL];
    __shared__ __attribute__((aligned(16))) unsigned char stage3[2 * PANEL];
    __shared__ __attribute__((aligned(16))) unsigned char stage4[2 * PANEL];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1, l32 = lane & 31, lhi = lane >> 5;
    // an XCD takes neighbouring tiles of the same tokens: they share panels in its L2
    const int64_t w = blockIdx.x, items = g.total * g.parts, per_xcd = (items + 7) / 8;
    const int64_t item = (w & 7) * per_xcd + (w >> 3);
    if ((w >> 3) >= per_xcd || item >= items) return;
    const int part = (int)(item / g.total);
    const int64_t L = item - part * g.total;
    int bi, bj;
    syrk_tile_of(g.nt, L, bi, bj);
    const int64_t trip0 = g.trips * part / g.parts, trip1 = g.trips * (part + 1) / g.parts;
    const int64_t r0 = (int64_t)bi * TILE, c0 = (int64_t)bj * TILE;

    // A copy is 1 KB: RPC token rows; a lane takes 16 bytes, chunk (position ^ swizzle of the token).  Wavefront w copies rows RPC (w COPIES + i) ..
    // of both panels.
    const int lrow = lane / (ROW / 16), pos = lane % (ROW / 16);
    const uint16_t* srcA[COPIES];
    const uint16_t* srcB[COPIES];
    int rowi[COPIES];
#pragma unroll
    for (int i = 0; i < COPIES; ++i) {
        rowi[i] = RPC * (wave * COPIES + i) + lrow;
        const int chunk = pos ^ (4 * (rowi[i] & 3));
        srcA[i] = g.X + min(r0 + 8 * chunk, g.n - 8);        // channels past n repeat the last ones: they only feed outputs that are not stored
        srcB[i] = g.X + min(c0 + 8 * chunk, g.n - 8);
    }
    const uint16_t* const zero = reinterpret_cast<const uint16_t*>(token_zeros);
    const int64_t first = trip0 * TRIP * STEP, last = trip1 * TRIP * STEP;           // this part's tokens (past t: zeros)
    auto issue_copies = [&](unsigned char* stage, int64_t token) {
        unsigned char* base = stage + wave * COPIES * 1024;
        token = min(token, last - STEP);                     // past the last step the copies repeat it, into a stage nobody multiplies
#pragma unroll
        for (int i = 0; i < COPIES; ++i) {
            const int64_t tk = token + rowi[i];
            const bool in = tk < g.t;
            const uint16_t* a = in ? srcA[i] + tk * g.ldx : zero;
            const uint16_t* b = in ? srcB[i] + tk * g.ldx : zero;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)a, (__attribute__((address_space(3))) void*)(base + i * 1024), 16, 0, 0);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)b, (__attribute__((address_space(3))) void*)(base + PANEL + i * 1024), 16, 0, 0);
        }
    };

    floatx16 acc[WT][WT];
#pragma unroll
    for (int s = 0; s < WT; ++s)
#pragma unroll
        for (int u = 0; u < WT; ++u)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[s][u][i] = 0.f;
    // Operands of 16 tokens (half kk of a step): lane l32 is the channel, tokens 16 kk + 8 lhi + 0 .. 7 as two transposed reads of four.
    // Of the 16 lanes that share a read lane i supplies token i / 4, channels 4 (i % 4) ..
    const int i16 = lane & 15, ch16 = (lane >> 4) & 1;
    const int tq = i16 >> 2;                                 // token & 3 of the address this lane supplies
    const int rdrow = (8 * lhi + tq) * ROW;
    auto rdoff = [&](int block, int s) {                     // block: first channel of the wavefront's tile / 32
        const int chunk = ((block + s) * 32 + 16 * ch16 + 4 * (i16 & 3)) / 8;
        return rdrow + ((chunk ^ (4 * tq)) << 4) + ((i16 & 1) << 3);
    };
    int offA[WT], offB[WT];
#pragma unroll
    for (int s = 0; s < WT; ++s) { offA[s] = rdoff(wm * WT, s); offB[s] = PANEL + rdoff(wn * WT, s); }
    uint4 fa[2][WT], fb[2][WT];
    auto turned = [&](const unsigned char* p) {
        typedef __attribute__((address_space(3))) shortx4* lds_short4;
        const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4)(p));
        const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4)(p + 4 * ROW));
        const uint2 a = __builtin_bit_cast(uint2, lo), b = __builtin_bit_cast(uint2, hi);
        return make_uint4(a.x, a.y, b.x, b.y);
    };
    auto fetch = [&](const unsigned char* st, int kk) {
#pragma unroll
        for (int s = 0; s < WT; ++s) {
            fa[kk][s] = turned(st + kk * (16 * ROW) + offA[s]);
            fb[kk][s] = turned(st + kk * (16 * ROW) + offB[s]);
        }
    };
    auto mma = [&](const uint4& a, const uint4& b, floatx16 c) {
        if constexpr (BF16) return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
        else return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(halfx8, a), __builtin_bit_cast(halfx8, b), c, 0, 0, 0);
    };
    auto half = [&](int kk) {
#pragma unroll
        for (int s = 0; s < WT; ++s)
#pragma unroll
            for (int u = 0; u < WT; ++u) acc[s][u] = mma(fa[kk][s], fb[kk][u], acc[s][u]);
        // LDS reads and copies between the matrix instructions
        constexpr int N = WT * WT, READS = 4 * WT, CP = COPIES;      // of this half
#pragma unroll
        for (int i = 0; i < N; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, READS / N > 0 ? READS / N : 1, 0);
            if (i % (N / CP > 0 ? N / CP : 1) == 0) __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
        }
    };
    auto next_stage = [&](unsigned char* refill, int64_t token, const unsigned char* cur, const unsigned char* nxt) {
        if constexpr (COPIES == 4) __builtin_amdgcn_s_waitcnt(0x4F70);          // vmcnt(16): the copies of the two steps after the next
        else __builtin_amdgcn_s_waitcnt(0x0F78);                                 // vmcnt(8)
        asm volatile("s_barrier" ::: "memory");              // the next step's stage is complete; everybody left `refill`
        issue_copies(refill, token);
        fetch(cur, 1);
        half(0);
        fetch(nxt, 0);
        half(1);
    };
    issue_copies(stage0, first);
    issue_copies(stage1, first + STEP);
    issue_copies(stage2, first + 2 * STEP);
    issue_copies(stage3, first + 3 * STEP);
    if constexpr (COPIES == 4) __builtin_amdgcn_s_waitcnt(0x4F78);              // vmcnt(24): step 0 has landed
    else __builtin_amdgcn_s_waitcnt(0x0F7C);                                     // vmcnt(12)
    asm volatile("s_barrier" ::: "memory");
    fetch(stage0, 0);
    // What keeps a long sum exact is short chains: the small tile, which has the registers, adds up every FLUSH trips apart.
    constexpr int FLUSH = 5;
    constexpr bool TWO = WT == 2;
    floatx16 sum[TWO ? WT : 1][TWO ? WT : 1];
    if constexpr (TWO) {
#pragma unroll
        for (int s = 0; s < WT; ++s)
#pragma unroll
            for (int u = 0; u < WT; ++u)
#pragma unroll
                for (int i = 0; i < 16; ++i) sum[s][u][i] = 0.f;
    }
    int left = FLUSH;
    for (int64_t k = first; k < last; k += TRIP * STEP) {
        if constexpr (TWO) {
            if (left == 0) {
#pragma unroll
                for (int s = 0; s < WT; ++s)
#pragma unroll
                    for (int u = 0; u < WT; ++u) {
                        sum[s][u] += acc[s][u];
#pragma unroll
                        for (int i = 0; i < 16; ++i) acc[s][u][i] = 0.f;
                    }
                left = FLUSH;
            }
            --left;
        }
        next_stage(stage4, k + 4 * STEP, stage0, stage1);
        next_stage(stage0, k + 5 * STEP, stage1, stage2);
        next_stage(stage1, k + 6 * STEP, stage2, stage3);
        next_stage(stage2, k + 7 * STEP, stage3, stage4);
        next_stage(stage3, k + 8 * STEP, stage4, stage0);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);                      // the surplus copies have landed before the workgroup ends
    if constexpr (TWO) {
#pragma unroll
        for (int s = 0; s < WT; ++s)
#pragma unroll
            for (int u = 0; u < WT; ++u) acc[s][u] += sum[s][u];
    }

    if (g.P) {
        float* pt = g.P + (L * g.parts + part) * (int64_t)(TILE * TILE);
#pragma unroll
        for (int s = 0; s < WT; ++s)
#pragma unroll
            for (int u = 0; u < WT; ++u) {
                float* pb = pt + (32 * (wm * WT + s) + 4 * lhi) * TILE + 32 * (wn * WT + u) + l32;
#pragma unroll
                for (int i = 0; i < 16; ++i) pb[(8 * (i >> 2) + (i & 3)) * TILE] = acc[s][u][i];
            }
        return;
    }
#pragma unroll
    for (int s = 0; s < WT; ++s)
#pragma unroll
        for (int u = 0; u < WT; ++u) {
            const int64_t col = c0 + 32 * (wn * WT + u) + l32, rbase = r0 + 32 * (wm * WT + s) + 4 * lhi;
            if (col >= g.n) continue;
            float* hb = g.H + rbase * g.ldh + col;
            // one owner per element in the launch: the memory system's float add is the same add as a load-add-store
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (rbase + 8 * (i >> 2) + (i & 3) < g.n) unsafeAtomicAdd(hb + (int64_t)(8 * (i >> 2) + (i & 3)) * g.ldh, 2.0f * acc[s][u][i]);
        }
}

// H tile += 2 (part 0 + part 1 + ..), in the order of the token ranges, eight at a time, then eight of these, then the sixty-fours: few channels have up
// to 512 parts, and 64 sums of eight one behind the other round each at the size of all before it.  A thread takes four columns.
template <int TILE>
__global__ __launch_bounds__(256) void tokens_reduce_kernel(TokenArgs g) {
    int bi, bj;
    syrk_tile_of(g.nt, (int64_t)blockIdx.x, bi, bj);
    const int e = ((int)blockIdx.y * 256 + (int)threadIdx.x) * 4, rt = e / TILE, ct = e % TILE;
    const float4* p = reinterpret_cast<const float4*>(g.P + (int64_t)blockIdx.x * g.parts * (TILE * TILE) + e);
    float4 sum = make_float4(0.f, 0.f, 0.f, 0.f), eights = sum;
    for (int q0 = 0; q0 < g.parts; q0 += 8) {
        float4 v[8], eight = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (q0 + q < g.parts) v[q] = p[(int64_t)(q0 + q) * (TILE * TILE / 4)];
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (q0 + q < g.parts) { eight.x += v[q].x; eight.y += v[q].y; eight.z += v[q].z; eight.w += v[q].w; }
        eights.x += eight.x; eights.y += eight.y; eights.z += eight.z; eights.w += eight.w;
        if ((q0 & 56) == 56 || q0 + 8 >= g.parts) {
            sum.x += eights.x; sum.y += eights.y; sum.z += eights.z; sum.w += eights.w;
            eights = make_float4(0.f, 0.f, 0.f, 0.f);
        }
    }
    const int64_t row = (int64_t)bi * TILE + rt, col = (int64_t)bj * TILE + ct;
    if (row >= g.n) return;
    float* h = g.H + row * g.ldh + col;
    const float s4[4] = {sum.x, sum.y, sum.z, sum.w};
#pragma unroll
    for (int c = 0; c < 4; ++c)
        if (col + c < g.n) h[c] += 2.0f * s4[c];
}

template <int WT>
int launch_tile(const TokenArgs& g, bool bf16, hipStream_t s) {
    constexpr int TILE = 64 * WT;
    const int64_t blocks = ceil_div(g.total * g.parts, 8) * 8;
    if (blocks > 0x7fffffffLL) return fail(GPTQ_ERR_UNSUPPORTED, "hessian: too many tiles");
    if (bf16) hipLaunchKernelGGL((syrk_tokens_kernel<true, WT>), dim3((unsigned)blocks), dim3(256), 0, s, g);
    else hipLaunchKernelGGL((syrk_tokens_kernel<false, WT>), dim3((unsigned)blocks), dim3(256), 0, s, g);
    GPTQ_LAUNCH_CHECK();
    if (g.P) {
        hipLaunchKernelGGL((tokens_reduce_kernel<TILE>), dim3((unsigned)g.total, TILE * TILE / 1024), dim3(256), 0, s, g);
        GPTQ_LAUNCH_CHECK();
    }
    return GPTQ_OK;
}

}  // namespace

int launch_syrk_tokens(float* H, int64_t ldh, const void* X, bool bf16, int64_t n, int64_t t, int64_t ldx, const TokenPlan& plan, void* ws, hipStream_t s) {
    TokenArgs g{};
    g.H = H; g.ldh = ldh; g.X = static_cast<const uint16_t*>(X); g.ldx = ldx; g.n = n; g.t = t;
    g.nt = (int)ceil_div(n, plan.tile);
    g.total = syrk_total_tiles(g.nt);
    g.parts = plan.parts;
    g.trips = ceil_div(t, TRIP * STEP);
    g.P = plan.parts > 1 ? static_cast<float*>(ws) : nullptr;
    return plan.tile == 256 ? launch_tile<4>(g, bf16, s) : launch_tile<2>(g, bf16, s);
}

}  // namespace gptq
