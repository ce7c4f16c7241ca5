// Scores of the router step written to memory: s = sigmoid(W_r x) (Sec. 2.2)
// as a plain tiled contraction, for batches too small to fill the chip with
// the fused kernel's 128-token tiles (router.hip); the selection then reads
// them back (select.hip).
//
// A small batch is bound by latency: the fused kernel runs one 128 x 384 tile
// per CU whatever T is, so 32 tokens cost as much contraction time as 16384
// (36.9 us at d = 2048, E = 768, two workgroups busy).  Here the tile shrinks
// with the batch until the launch has about as many workgroups as the chip has
// CUs, and each wave keeps D chunks of both operands in flight in registers:
// 4.9 us at T = 32 (5.4 us with each chunk's operands read from LDS after it is
// staged), 12.9 us for T = 777, d = 4096, E = 256 row-major (fused: 92.6 us with
// 128 x 256 tiles), 7.4 us for fp32 T = 4096, d = 256, E = 64 (fused: 29.4 us).
// The score matrix of such a batch is small enough to stay in L2 and the
// Infinity Cache between the two launches.
//
// Accumulation order: one wave sums a score over k in chunk order with the same
// MFMA shape as the fused tiling of the same pool (16x16x32 or 32x32x16, fp32
// 32x32x2), never splitting k, so a token's scores have the same bits whichever
// path its batch takes.
#include "common.h"
#include "internal.h"

#include <type_traits>

#pragma clang fp contract(off)

namespace idb {

namespace {

constexpr int kEnough16 = 160;  // workgroups that occupy enough of the 256 CUs (16x16 tiles;
constexpr int kEnough32 = 120;  // 32x32 tiles, whose next smaller choice is a single block)
constexpr int kFull = 224;      // workgroups of the largest tile, which needs nearly a whole round
constexpr int kScoreRow = 160;  // LDS bytes per staged token row (128 + 32 pad)

// M32: 32x32 MFMA blocks (else 16x16); TB token blocks per workgroup, shared by
// the waves through LDS; EB expert blocks per wave; D chunks in flight (even).
template <bool M32, bool F32, int WAVES, int TB, int EB, int D>
struct ScoreCfg {
    static constexpr int NT = WAVES * 64;
    static constexpr int MB = M32 ? 32 : 16;
    static constexpr int BT = MB * TB;
    static constexpr int WE = MB * EB;
    static constexpr int BE = WAVES * WE;
    static constexpr int PPT = (BT * 8 + NT - 1) / NT;  // 16-byte token-tile pieces per thread per chunk
    static constexpr int UNITS = M32 ? 4 : 2;           // A operands of an expert block per chunk
    static constexpr int STAGE = BT * kScoreRow;
    static_assert(D % 2 == 0, "the LDS stage of a register set is fixed");
    static_assert(!F32 || M32, "fp32 inputs use 32x32x2 MFMAs");
};

template <bool M32, bool F32, bool PACKED, int WAVES, int TB, int EB, int D>
__global__ __launch_bounds__(WAVES * 64) void score_kernel(RouterArgs a, int NS, float* __restrict__ scores) {
    using C = ScoreCfg<M32, F32, WAVES, TB, EB, D>;
    using Acc = typename std::conditional<M32, floatx16, floatx4>::type;
    constexpr int NR = M32 ? 16 : 4;
    __shared__ __attribute__((aligned(16))) unsigned char smem[2 * C::STAGE];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & (C::MB - 1), lg = lane / C::MB;  // row of a block, k group
    const int L = xcd_block_order();
    const int tile = L / NS;
    const int slice = L - tile * NS;

    const int64_t T = a.T;
    const int E = a.E;
    const int64_t tok0 = (int64_t)tile * C::BT;
    const int e_wave0 = slice * C::BE + wave * C::WE;
    const int64_t RB = (int64_t)a.d * (F32 ? 4 : 2);
    const int NCH = (int)(RB / 128);

    // the selection that follows counts into these
    if (a.zero_counts && blockIdx.x == 0)
        for (int e = tid; e < E; e += C::NT) a.counts[e] = 0;
    if (a.ticket && blockIdx.x == 0 && tid == 0) *a.ticket = 0u;

    // A operands (router rows), 16 bytes per lane.  16x16: unit s of chunk c is
    // row lr, bytes c*128 + 64 s + 16 lg.  32x32: unit u is row lr, bytes
    // c*128 + 64 lg + 16 u.  Packed: see pack_weight_kernel (router.hip).
    constexpr int WU = M32 ? (PACKED ? 256 : 16) : (PACKED ? 1024 : 64);
    constexpr int WCH = PACKED ? 2048 : 128;
    const __amdgpu_buffer_rsrc_t wres = make_rsrc(a.W, (int64_t)E * RB);
    const int wvoff = M32 ? (PACKED ? (lr >> 4) * NCH * 2048 + lg * 1024 + (lr & 15) * 16 : lr * (int)RB + 64 * lg)
                          : (PACKED ? lane * 16 : lr * (int)RB + 16 * lg);
    int wsoff[EB];
#pragma unroll
    for (int eb = 0; eb < EB; ++eb) {
        int blk = e_wave0 / C::MB + eb;
        blk = blk < E / C::MB ? blk : E / C::MB - 1;  // padding blocks read a valid block; never stored
        wsoff[eb] = PACKED ? blk * NCH * (128 * C::MB) : blk * C::MB * (int)RB;
    }
    // Token-tile pieces: piece p = tid + NT*q covers row (p/8) mod BT, bytes
    // 16*(p%8) of the chunk (pieces past the tile repeat one of it).  Rows past
    // T re-read row T-1 (never stored).
    const int nrows = (int)((T - tok0) < C::BT ? (T - tok0) : C::BT);
    const __amdgpu_buffer_rsrc_t xres =
        make_rsrc(reinterpret_cast<const char*>(a.x) + tok0 * RB, (int64_t)nrows * RB);
    int xvoff[C::PPT];
    int xdst[C::PPT];
#pragma unroll
    for (int q = 0; q < C::PPT; ++q) {
        const int p = tid + C::NT * q;
        const int row = (p >> 3) & (C::BT - 1), c16 = p & 7;
        const int rowc = row < nrows ? row : nrows - 1;
        xvoff[q] = rowc * (int)RB + c16 * 16;
        xdst[q] = row * kScoreRow + c16 * 16;
    }
    static_assert((C::BT & (C::BT - 1)) == 0, "rows wrap by a mask");
    const int boff = lr * kScoreRow + (M32 ? 64 : 16) * lg;

    Acc acc[TB][EB];
#pragma unroll
    for (int tb = 0; tb < TB; ++tb)
#pragma unroll
        for (int eb = 0; eb < EB; ++eb)
#pragma unroll
            for (int r = 0; r < NR; ++r) acc[tb][eb][r] = 0.0f;

    // Register set j holds chunk c = j (mod D) of both operands from D chunks
    // ahead; the token tile passes through two LDS stages.  The main loop takes
    // whole groups of D chunks without a branch (prefetch targets are clamped
    // to the last chunk) and the rest is peeled after it: a conditional exit
    // inside the group would merge into the loop's head and make its waits
    // drain the queue every D chunks (measured: 21.5 us per launch either with
    // D = 4 or 8 at T = 4096, d = 2048, E = 768).
    uint4 w[D][EB][C::UNITS], xr[D][C::PPT];
    auto load_x = [&](int c, int j) {
#pragma unroll
        for (int q = 0; q < C::PPT; ++q) xr[j][q] = bload16(xres, xvoff[q], c * 128);
    };
    auto store_x = [&](int stage, int j) {
#pragma unroll
        for (int q = 0; q < C::PPT; ++q) *reinterpret_cast<uint4*>(smem + stage * C::STAGE + xdst[q]) = xr[j][q];
    };
    const int last = NCH - 1;
#pragma unroll
    for (int j = 0; j < D; ++j) {
        const int c = j < last ? j : last;
        load_x(c, j);
#pragma unroll
        for (int eb = 0; eb < EB; ++eb)
#pragma unroll
            for (int u = 0; u < C::UNITS; ++u) w[j][eb][u] = bload16(wres, wvoff + WU * u, wsoff[eb] + c * WCH);
    }
    store_x(0, 0);
    __syncthreads();
    auto read_x = [&](int stage, uint4 (&bx)[C::UNITS][TB], int u) {
        const unsigned char* st = smem + stage * C::STAGE + boff;
#pragma unroll
        for (int tb = 0; tb < TB; ++tb)
            bx[u][tb] = *reinterpret_cast<const uint4*>(st + tb * C::MB * kScoreRow + (M32 ? 16 : 64) * u);
    };
    auto mfma = [&](int j, const uint4 (&bx)[C::UNITS][TB], int u, bool prefetch, int cn) {
#pragma unroll
        for (int tb = 0; tb < TB; ++tb)
#pragma unroll
            for (int eb = 0; eb < EB; ++eb) {
                if constexpr (M32) acc[tb][eb] = mfma_unit<F32>(w[j][eb][u], bx[u][tb], acc[tb][eb]);
                else
                    acc[tb][eb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(w[j][eb][u]),
                                                                          as_bf16x8(bx[u][tb]), acc[tb][eb], 0, 0, 0);
            }
        if (prefetch) {
#pragma unroll
            for (int eb = 0; eb < EB; ++eb) w[j][eb][u] = bload16(wres, wvoff + WU * u, wsoff[eb] + cn * WCH);
        }
    };
    // One chunk, and the next one's tokens into the other stage.  A wave alone
    // needs no barrier (its LDS accesses execute in order): it stages the next
    // chunk and reads all its operands back before this one's MFMAs, which
    // cover the round trip; nothing else on its SIMD would.
    uint4 bq[WAVES == 1 ? 2 : 1][C::UNITS][TB];
    if constexpr (WAVES == 1) {
#pragma unroll
        for (int u = 0; u < C::UNITS; ++u) read_x(0, bq[0], u);
    }
    auto step = [&](int j, bool prefetch, int cn) {
        if constexpr (WAVES == 1) {
            store_x((j + 1) & 1, (j + 1) % D);
            wave_sync();
#pragma unroll
            for (int u = 0; u < C::UNITS; ++u) read_x((j + 1) & 1, bq[(j + 1) & 1], u);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < C::UNITS; ++u) mfma(j, bq[j & 1], u, prefetch, cn);
        } else {
#pragma unroll
            for (int u = 0; u < C::UNITS; ++u) {
                read_x(j & 1, bq[0], u);
                mfma(j, bq[0], u, prefetch, cn);
            }
            store_x((j + 1) & 1, (j + 1) % D);
            __syncthreads();
        }
    };
    int c0 = 0;
    for (; c0 + D <= NCH; c0 += D) {
#pragma unroll
        for (int j = 0; j < D; ++j) {
            const int cn = c0 + j + D < last ? c0 + j + D : last;
            load_x(cn, j);
            step(j, true, cn);
        }
    }
#pragma unroll
    for (int j = 0; j + 1 < D; ++j) {
        if (c0 + j < NCH) step(j, false, 0);
    }

    // MFMA output layouts: 16x16 - lane (lr, lg) holds token lr, experts 4 lg + r;
    // 32x32 - token lr, experts 8 (r/4) + 4 lg + r%4.
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
        const int64_t tok = tok0 + tb * C::MB + lr;
        if (tok < T) {
#pragma unroll
            for (int eb = 0; eb < EB; ++eb) {
                const int e0 = e_wave0 + eb * C::MB;
                if (e0 < E) {
#pragma unroll
                    for (int r4 = 0; r4 < NR / 4; ++r4) {
                        const float4 s4 =
                            make_float4(sigmoid_fast(acc[tb][eb][4 * r4]), sigmoid_fast(acc[tb][eb][4 * r4 + 1]),
                                        sigmoid_fast(acc[tb][eb][4 * r4 + 2]), sigmoid_fast(acc[tb][eb][4 * r4 + 3]));
                        const int64_t at = tok * E + e0 + 8 * r4 + 4 * lg;
                        *reinterpret_cast<float4*>(scores + at) = s4;
                        if (a.dump) *reinterpret_cast<float4*>(a.dump + at) = s4;
                    }
                }
            }
        }
    }
}

template <bool M32, bool F32, int WAVES, int TB, int EB, int D>
hipError_t launch_scores_cfg(const RouterArgs& a, float* scores, hipStream_t stream) {
    using C = ScoreCfg<M32, F32, WAVES, TB, EB, D>;
    const int NS = (a.E + C::BE - 1) / C::BE;
    const int64_t blocks = (a.T + C::BT - 1) / C::BT * NS;
    if (a.w_packed)
        hipLaunchKernelGGL((score_kernel<M32, F32, true, WAVES, TB, EB, D>), dim3((unsigned)blocks), dim3(C::NT), 0,
                           stream, a, NS, scores);
    else
        hipLaunchKernelGGL((score_kernel<M32, F32, false, WAVES, TB, EB, D>), dim3((unsigned)blocks), dim3(C::NT), 0,
                           stream, a, NS, scores);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_scores(const RouterTiling& t, const RouterArgs& a, float* scores, hipStream_t stream) {
    // The largest tile that still gives the chip enough workgroups.  A larger
    // tile reads fewer operand bytes through L2 per score (what bounds these
    // launches once the chip is full), a smaller one fills more CUs.  us per
    // launch at d = 2048, E = 768 (16x16; 64 x 192, 64 x 128, 64 x 64, one 16 x 16
    // block per wave): T = 4096 19.3, 22.1, 23.1, -; T = 2048 17.7, 14.8, 16.1, -;
    // T = 1024 -, -, 11.3, -; T = 256 -, -, 7.6 (32 x 64), 7.3; T = 32 -, -, 6.1
    // (16 x 64), 4.9.  32x32 at d = 1024, E = 1024, T = 5003: 64 x 128 20.4, 64 x 256
    // 24.4, 128 x 256 21.6, 32 x 128 26.1; at d = 4096, E = 256, T = 777: one block
    // per wave 11.9, 32 x 128 15.5, 64 x 128 19.8.
    auto blocks = [&](int bt, int be) { return (a.T + bt - 1) / bt * ((a.E + be - 1) / be); };
    if (t.is_f32) return launch_scores_cfg<true, true, 1, 1, 1, 8>(a, scores, stream);
    if (!tiling_is_16(t)) {
        if (blocks(64, 128) >= kEnough32) return launch_scores_cfg<true, false, 4, 2, 1, 4>(a, scores, stream);
        return launch_scores_cfg<true, false, 1, 1, 1, 8>(a, scores, stream);
    }
    if (blocks(128, 384) >= kFull) return launch_scores_cfg<false, false, 8, 8, 3, 2>(a, scores, stream);
    if (blocks(64, 192) >= kEnough16) return launch_scores_cfg<false, false, 4, 4, 3, 4>(a, scores, stream);
    if (blocks(64, 128) >= kEnough16) return launch_scores_cfg<false, false, 4, 4, 2, 4>(a, scores, stream);
    if (blocks(64, 64) >= kEnough16) return launch_scores_cfg<false, false, 4, 4, 1, 4>(a, scores, stream);
    return launch_scores_cfg<false, false, 1, 1, 1, 8>(a, scores, stream);
}

}  // namespace idb
