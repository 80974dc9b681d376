// Step 1 for layers of few channels, X read in place (channel-major, no workspace): H += 2 X X^T.
//
// A matrix of few tiles leaves most of the chip idle and walks all tokens in one long chain per tile (256 channels:
// 2 tiles of 256 x 128 on 256 CUs, 4096 float32 tokens in 471 us).  Here the tile is small -- T x T, T = 64, 32 or 16 -- and the
// wavefronts of a workgroup share the tokens of ONE tile: wavefront w multiplies chunks w, w + WAVES, .. of CHUNK tokens,
// the next chunk's operands on their way while this one is multiplied, and
// the partial tiles are added through LDS in a fixed order, so a call gives the same bits every time.
// Bound: the vector cache.  A matrix operand has a different row in every neighbouring lane, so a load straight into registers touches
// 16 rows x 64 bytes, half cache lines, and moves ~20 bytes per cycle and CU.  So a wavefront copies whole lines of its chunk, 8
// rows x 128 bytes an instruction, into LDS of its own and takes the operands from there; the order of the sums, and the bits, are the same.
// Measured, us, straight / through LDS: float16 256 channels x 4096 tokens 11.8 / 6.2, 512 x 16384 62 / 26, 1000 x 16384 117 / 51, 1536 x 16384
// 234 / 115 (350 TFLOP/s on its whole tiles' flops); float32 256 x 4096 19.3 / 13.1, 352 x 16384 62 / 41.  Straight stays the float32 tiles of 32 and
// 64 (512 x 16384 140 / 153, 1000 x 16384 478 / 571: they are held by the float32 instructions, one chunk in LDS is too little ahead), and calls of
// up to three chunks, most of them their own latency (1536 x 128 9.1 / 9.7, x 64 7.8 / 9.0, x 256 12.5 / 10.2).
#include "hessian_small.h"

namespace gptq {

typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

namespace {

struct SmallArgs { float* H; int64_t ldh; const void* X; int64_t ldx, n, t; };

// TYPE: GPTQ_F16, GPTQ_BF16 or GPTQ_F32.  CHAINS: sums that a wavefront's chunks go to in turn; the sums are added in the order of their
// first chunks, so that 8 wavefronts of two give the bits of 16 of one.
template <int TYPE, int T, int WAVES, int CHAINS = 1>
__global__ __launch_bounds__(64 * WAVES) void syrk_small_kernel(SmallArgs g) {
    constexpr int SZ = TYPE == GPTQ_F32 ? 4 : 2;
    constexpr int EL = 16 / SZ;                              // tokens per load
    constexpr int PER = 2;                                   // loads of a row per chunk
    constexpr int CHUNK = PER * 4 * EL;                      // 64 tokens, or 32 of float32
    constexpr int S = T / 16;                                // 16 x 16 tiles per side
    constexpr int SLOT = T * T * 4;
    constexpr bool THROUGH_LDS = SZ == 2 || T == 16;
    constexpr int U = T == 16 ? 2 : 1;                       // chunks of a wavefront that are copied at a time
    constexpr int OPERAND = T * 128, STAGE = THROUGH_LDS ? U * 2 * OPERAND : SLOT;    // 128 bytes of T rows; A and B
    static_assert(SLOT <= STAGE, "the partial tiles take the place of the operands");
    __shared__ __attribute__((aligned(16))) unsigned char lds[WAVES * STAGE];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, kq = lane >> 4;
    // tile of the upper triangle: column by column
    int bj = 0, bi = (int)blockIdx.x;
    while (bi > bj) { bi -= bj + 1; ++bj; }

    // Rows past n repeat the last one: they only feed outputs that are not stored.
    const char* base = static_cast<const char*>(g.X);
    auto row_at = [&](int64_t row) { return base + min(row, g.n - 1) * g.ldx * SZ; };
    const char* rowA[S];
    const char* rowB[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
        rowA[s] = row_at((int64_t)bi * T + 16 * s + l16) + kq * 16;
        rowB[s] = row_at((int64_t)bj * T + 16 * s + l16) + kq * 16;
    }
    // A copy moves 8 rows x 128 bytes, whole cache lines, lane l position l % 8 of row l / 8: the chunk (l % 8) ^ (row / 2 % 8), so that 16
    // rows at the same chunk, what 16 lanes of a read touch together, lie in different banks
    const char* srcA[2 * S];
    const char* srcB[2 * S];
#pragma unroll
    for (int j = 0; j < 2 * S; ++j) {
        const int r = 8 * j + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
        srcA[j] = row_at((int64_t)bi * T + r) + c * 16;
        srcB[j] = row_at((int64_t)bj * T + r) + c * 16;
    }
    unsigned char* const stage = lds + __builtin_amdgcn_readfirstlane(wave) * STAGE;
    auto copy = [&](int64_t chunk, int u) {
        const int64_t off = chunk * (CHUNK * SZ);
#pragma unroll
        for (int j = 0; j < 2 * S; ++j) {
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(srcA[j] + off),
                                             (__attribute__((address_space(3))) void*)(stage + 2 * u * OPERAND + j * 1024), 16, 0, 0);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(srcB[j] + off),
                                             (__attribute__((address_space(3))) void*)(stage + (2 * u + 1) * OPERAND + j * 1024), 16, 0, 0);
        }
    };
    uint4 a[2][S][PER], b[2][S][PER];
    auto fetch = [&]() {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int i = 0; i < PER; ++i) {
                    const int at = (16 * s + l16) * 128 + (((4 * i + kq) ^ ((l16 >> 1) & 7)) << 4);
                    a[u][s][i] = *reinterpret_cast<const uint4*>(stage + 2 * u * OPERAND + at);
                    b[u][s][i] = *reinterpret_cast<const uint4*>(stage + (2 * u + 1) * OPERAND + at);
                }
    };
    // ... or straight into registers: a whole chunk, no branch around it, so that the wait for one buffer does not wait for the other's loads
    auto load = [&](int64_t chunk, int buf) {
        const int64_t off = chunk * (CHUNK * SZ);
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                a[buf][s][i] = *reinterpret_cast<const uint4*>(rowA[s] + off + 64 * i);
                b[buf][s][i] = *reinterpret_cast<const uint4*>(rowB[s] + off + 64 * i);
            }
    };
    // The tokens past the last whole chunk, zeros past the last token: the 16 bytes that hold a lane's, or the last 16 that hold any, masked
    // -- without a branch, so that all loads are on their way at once (with one around each, 8 tokens of 2048 channels took 15.0 us; 13.5 through
    // the larger tiles).  What a row's last 16 bytes hold past its last token is in the row (its distance to the next is whole 16 bytes) but
    // for the last row's: the 16 rows with it are taken element by element.
    auto load_tail = [&](const char* row, int64_t k0, uint4 (&d)[PER]) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int64_t k = k0 + (4 * i + kq) * EL;
            const uint4 v = *reinterpret_cast<const uint4*>(row - kq * 16 + min(k, (g.t - 1) / EL * EL) * SZ);
            const int64_t left = g.t - k;
            auto keep = [&](uint32_t w, int j) {             // word j of the 16 bytes
                if constexpr (SZ == 4) return left > j ? w : 0u;
                else return left >= 2 * j + 2 ? w : left == 2 * j + 1 ? w & 0xFFFFu : 0u;
            };
            d[i] = make_uint4(keep(v.x, 0), keep(v.y, 1), keep(v.z, 2), keep(v.w, 3));
        }
    };
    auto load_tail_of_last_row = [&](const char* row, int64_t k0, uint4 (&d)[PER]) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int64_t k = k0 + (4 * i + kq) * EL;
            const char* p = row + k0 * SZ + 64 * i;
            if (k + EL <= g.t) { d[i] = *reinterpret_cast<const uint4*>(p); continue; }
            uint32_t w[4] = {0u, 0u, 0u, 0u};
            if (k < g.t) {
#pragma unroll
                for (int e = 0; e < EL - 1; ++e) {
                    if (k + e < g.t) {
                        if constexpr (SZ == 4) w[e] = reinterpret_cast<const uint32_t*>(p)[e];
                        else w[e >> 1] |= (uint32_t)reinterpret_cast<const uint16_t*>(p)[e] << (16 * (e & 1));
                    }
                }
            }
            d[i] = make_uint4(w[0], w[1], w[2], w[3]);
        }
    };
    floatx4 sums[CHAINS][S][S];
#pragma unroll
    for (int h = 0; h < CHAINS; ++h)
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int u = 0; u < S; ++u)
#pragma unroll
                for (int i = 0; i < 4; ++i) sums[h][s][u][i] = 0.f;
    auto products = [&](floatx4 (&acc)[S][S], const uint4 (&x)[S][PER], const uint4 (&y)[S][PER]) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if constexpr (TYPE == GPTQ_F32) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int s = 0; s < S; ++s)
#pragma unroll
                        for (int u = 0; u < S; ++u) {
                            const uint32_t xa[4] = {x[s][i].x, x[s][i].y, x[s][i].z, x[s][i].w}, yb[4] = {y[u][i].x, y[u][i].y, y[u][i].z, y[u][i].w};
                            acc[s][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(xa[e]), __uint_as_float(yb[e]), acc[s][u], 0, 0, 0);
                        }
            } else {
#pragma unroll
                for (int s = 0; s < S; ++s)
#pragma unroll
                    for (int u = 0; u < S; ++u) {
                        if constexpr (TYPE == GPTQ_BF16)
                            acc[s][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x[s][i]), __builtin_bit_cast(bf16x8, y[u][i]), acc[s][u], 0, 0, 0);
                        else
                            acc[s][u] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(halfx8, x[s][i]), __builtin_bit_cast(halfx8, y[u][i]), acc[s][u], 0, 0, 0);
                    }
            }
        }
    };
    const int64_t chunks = g.t / CHUNK;
    constexpr int SHORT = 3;                                 // chunks of the calls that go straight all the same: a wavefront has one at most
    static_assert(SHORT < WAVES, "");
    const bool through_lds = THROUGH_LDS && chunks > SHORT;
    // A wavefront's copies are its own business, no barrier: it waits for them, takes the operands into registers, and has the next ones
    // on their way while it multiplies.  (Past its last chunk the last of all is copied again.)
    if (THROUGH_LDS && !through_lds && wave < chunks) {
        load(wave, 0);
        products(sums[0], a[0], b[0]);
    }
    if (!THROUGH_LDS && wave < chunks) {
        const int64_t last = chunks - 1;
        load(wave, 0);
        for (int64_t c = wave; c < chunks; c += 2 * WAVES) {
            load(min(c + WAVES, last), 1);
            __builtin_amdgcn_sched_barrier(0);
            products(sums[0], a[0], b[0]);
            if (c + WAVES >= chunks) break;
            __builtin_amdgcn_sched_barrier(0);
            load(min(c + 2 * WAVES, last), 0);
            __builtin_amdgcn_sched_barrier(0);
            products(sums[0], a[1], b[1]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if (through_lds && wave < chunks) {
        const int64_t last = chunks - 1;
#pragma unroll
        for (int u = 0; u < U; ++u) copy(min((int64_t)wave + u * WAVES, last), u);
        auto trip = [&](int64_t c, floatx4 (&acc)[S][S]) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            fetch();
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
            for (int u = 0; u < U; ++u) copy(min(c + (U + u) * WAVES, last), u);
            __builtin_amdgcn_sched_barrier(0);
            products(acc, a[0], b[0]);
            if (U > 1 && c + WAVES < chunks) products(acc, a[U - 1], b[U - 1]);
            __builtin_amdgcn_sched_barrier(0);
        };
        for (int64_t c = wave; c < chunks; c += CHAINS * U * WAVES) {
            trip(c, sums[0]);
            if (CHAINS > 1 && c + WAVES < chunks) trip(c + WAVES, sums[CHAINS - 1]);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    if (g.t % CHUNK != 0 && wave == WAVES - 1) {
        auto load_rows = [&](const char* row, int64_t first, uint4 (&d)[PER]) {
            if (first + 16 < g.n) load_tail(row, chunks * CHUNK, d);
            else if (first < g.n) load_tail_of_last_row(row, chunks * CHUNK, d);
            else {
#pragma unroll
                for (int i = 0; i < PER; ++i) d[i] = make_uint4(0u, 0u, 0u, 0u);
            }
        };
        if (g.t % EL == 0 || (int64_t)bj * T + T < g.n) {     // (rows lie above columns)
#pragma unroll
            for (int s = 0; s < S; ++s) {
                load_tail(rowA[s], chunks * CHUNK, a[0][s]);
                load_tail(rowB[s], chunks * CHUNK, b[0][s]);
            }
        } else {
#pragma unroll
            for (int s = 0; s < S; ++s) {
                load_rows(rowA[s], (int64_t)bi * T + 16 * s, a[0][s]);
                load_rows(rowB[s], (int64_t)bj * T + 16 * s, b[0][s]);
            }
        }
        products(sums[CHAINS - 1], a[0], b[0]);
    }
    if (through_lds) __syncthreads();                        // everybody has read the operands whose place the partial tiles take
    unsigned char* const part = lds;
    // every wavefront leaves its partial tile in LDS, then takes its share of the tile: the partial sums of an element are
    // added in the order of the wavefronts
    floatx4* mine = reinterpret_cast<floatx4*>(part + wave * SLOT);
    constexpr int SHARE = (S * S + WAVES - 1) / WAVES;
    floatx4 total[SHARE], old[SHARE];
    // 16 x 16 tile wave + i WAVES of this tile: rows row_of(i) + e, column col_of(i); H as it is is asked for before the sums are added
    auto mine_too = [&](int i) { return S * S % WAVES == 0 || wave + i * WAVES < S * S; };
    auto col_of = [&](int i) { return (int64_t)bj * T + 16 * ((wave + i * WAVES) % S) + l16; };
    auto row_of = [&](int i) { return (int64_t)bi * T + 16 * ((wave + i * WAVES) / S) + 4 * kq; };
#pragma unroll
    for (int i = 0; i < SHARE; ++i) {
        total[i] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 4; ++e)
            old[i][e] = mine_too(i) && col_of(i) < g.n && row_of(i) + e < g.n ? g.H[(row_of(i) + e) * g.ldh + col_of(i)] : 0.f;
    }
#pragma unroll
    for (int h = 0; h < CHAINS; ++h) {
        if (h > 0) __syncthreads();
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int u = 0; u < S; ++u) mine[(s * S + u) * 64 + lane] = sums[h][s][u];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < SHARE; ++i)
            if (mine_too(i)) {
#pragma unroll
                for (int w = 0; w < WAVES; ++w) total[i] += reinterpret_cast<const floatx4*>(part + w * SLOT)[(wave + i * WAVES) * 64 + lane];
            }
    }
#pragma unroll
    for (int i = 0; i < SHARE; ++i)
        if (mine_too(i) && col_of(i) < g.n) {
            float* h = g.H + row_of(i) * g.ldh + col_of(i);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (row_of(i) + e < g.n) h[e * g.ldh] = old[i][e] + 2.0f * total[i][e];
        }
}

template <int TYPE>
int launch(const SmallArgs& a, hipStream_t s) {
    const int64_t n64 = ceil_div(a.n, 64), n32 = ceil_div(a.n, 32);
    const int64_t n16 = ceil_div(a.n, 16);
    // The smallest tile while every CU has at most one: half the bytes a tile reads.  us, 16 x 16 / 32 x 32, both straight, float32 (float16): 4096 tokens of 64 channels
    // 18.7 / 37.2 (11.8 / 19.9), 352 19.9 / 39.5 (12.5 / 20.4), 400 35.6 / 39.7 (21.4 / 20.8), 512 52 / 40; 16384 of 352 61 / 141 (34 / 62), 400 118 / 141 (63 / 62).
    // Tiles of 64, 16-bit: as soon as those of 32 are more than one a CU (32 x 32 / 64 x 64: 8192 tokens of 712 28.2 / 26.7, 800 30.4 / 26.8, 960 36.8 / 27.9, 64 tokens of 900
    // 7.2 / 6.0; at 700, 253 tiles of 32, these are ahead).
    // (Up to 960 channels, where those of 32 have 16 wavefronts and an element's tokens 16 sums, with two sums a wavefront: the same bits.
    // With 8 sums 65536 tokens had a relative error of 1.8e-7, not 1.1e-7, 16384 one of 1.0e-7, not 0.8e-7; 8192 tokens of 960 take 30 us either way.)
    if constexpr (TYPE != GPTQ_F32) {
        if (n32 * (n32 + 1) / 2 > 256 && n64 * (n64 + 1) / 2 < 128) {
            hipLaunchKernelGGL((syrk_small_kernel<TYPE, 64, 8, 2>), dim3((unsigned)(n64 * (n64 + 1) / 2)), dim3(512), 0, s, a);
            GPTQ_LAUNCH_CHECK();
            return GPTQ_OK;
        }
    }
    if (n64 * (n64 + 1) / 2 >= 128) {
        hipLaunchKernelGGL((syrk_small_kernel<TYPE, 64, 8>), dim3((unsigned)(n64 * (n64 + 1) / 2)), dim3(512), 0, s, a);
    } else if (n16 * (n16 + 1) / 2 <= 256) {
        hipLaunchKernelGGL((syrk_small_kernel<TYPE, 16, 16>), dim3((unsigned)(n16 * (n16 + 1) / 2)), dim3(1024), 0, s, a);
    } else {
        hipLaunchKernelGGL((syrk_small_kernel<TYPE, 32, 16>), dim3((unsigned)(n32 * (n32 + 1) / 2)), dim3(1024), 0, s, a);
    }
    GPTQ_LAUNCH_CHECK();
    return GPTQ_OK;
}

}  // namespace

int launch_syrk_small(float* H, int64_t ldh, const void* X, int xdtype, int64_t n, int64_t t, int64_t ldx, hipStream_t s) {
    const SmallArgs a{H, ldh, X, ldx, n, t};
    if (xdtype == GPTQ_F32) return launch<GPTQ_F32>(a, s);
    if (xdtype == GPTQ_BF16) return launch<GPTQ_BF16>(a, s);
    return launch<GPTQ_F16>(a, s);
}

}  // namespace gptq
