// Bias-adjusted Top-K selection from given fp32 scores (Eq. pid-routing), gate
// weights from the unbiased scores (Sec. 2.2) and per-expert load counts
// (Eq. pid-error): the router step without the gate contraction, an HBM-bound
// pass over a materialised T x E score matrix.
//
// Two kernels:
//  * select_reg_kernel (E % 4 == 0, 16-byte aligned scores): 16 lanes (one DPP
//    row) per token, each holding every 16th float4 of the row in registers.
//    The K-th largest of the row's 16 G group maxima (G = 1, 2 or 4 groups per
//    lane) is a lower bound tau of the token's K-th largest biased score; only
//    the float4 chunks whose maximum reaches tau are read again, and their
//    values >= tau go to a short LDS list whose entries are ranked by counting.
//    A token whose list would overflow takes K exact argmax rounds over its row
//    instead.  G grows with K so that the list stays short: K of 16 G groups
//    holding K or more values gives about 16 G ln(1 / (1 - K / 16 G)) of them
//    (16 at K = 10, G = 1; 22 at K = 16, G = 2; 44 at K = 32, G = 4), and with
//    G = 1 every list overflows from K = 16 on.  It also ends the router's
//    scored path, where its last workgroup applies the controller update.
//  * select_kernel (other row lengths and alignments): a workgroup of 512 threads walks tiles
//    of 32 tokens (grid-stride, one workgroup per CU: the score rows of a tile
//    take most of the LDS).  A tile's scores go from registers into the LDS
//    score rows of the selection epilogue (epilogue.h, one slice of BE >= E
//    experts, padding -inf); right after, the next tile's scores are loaded
//    into the same registers, so their HBM reads overlap the selection of the
//    current tile.
// Both flush their LDS histogram once per workgroup.
#include "common.h"
#include "controller_block.h"
#include "epilogue.h"
#include "internal.h"

#include <utility>

#pragma clang fp contract(off)

namespace idb {

namespace {

constexpr int kSelThreads = 512;
constexpr int kSelTile = 32;  // tokens per tile
// LDS for a tile's score rows: 32 rows of 1028 floats at BE = 1024 (131.6 KB);
// the epilogue's other arrays fit in the remaining 29 KB of the 160 KB.
constexpr int kSelScoreLds = 160 * 1024 - 29 * 1024;

__global__ void fill_i32_kernel(int32_t* p, int32_t value, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = value;
}

// BE: the slice width (a multiple of 256 >= E).
template <int BE>
__global__ __launch_bounds__(kSelThreads) void select_kernel(RouterArgs a, const float* __restrict__ scores) {
    using EC = EpiCfg<kSelThreads, kSelTile, BE, 0, kSelScoreLds>;
    static_assert(EC::NPASS == 1, "one pass per tile");
    __shared__ __attribute__((aligned(16))) unsigned char smem[EC::LDS];
    constexpr int PIECES = kSelTile * BE / 4;      // pieces of four scores of a tile
    constexpr int PER = PIECES / kSelThreads;      // per thread
    static_assert(PER * kSelThreads == PIECES, "tile pieces split evenly");
    const int tid = threadIdx.x;
    const int64_t T = a.T;
    const int E = a.E;

    float breg[EC::NBIAS];
    prefetch_bias<EC>(a, 0, breg);
    epi_begin<EC>(smem, breg);

    // piece p = tid + kSelThreads * i: tile row p / (BE/4), columns 4 (p % (BE/4)) + c
    float4 r[PER];
    auto load = [&](int64_t tile) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int p = tid + kSelThreads * i;
            const int row = p / (BE / 4), c4 = 4 * (p % (BE / 4));
            const int64_t t = tile * kSelTile + row;
            float4 f = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
            if (t < T) {
                const float* src = scores + t * (int64_t)E + c4;
                if (c4 + 0 < E) f.x = src[0];
                if (c4 + 1 < E) f.y = src[1];
                if (c4 + 2 < E) f.z = src[2];
                if (c4 + 3 < E) f.w = src[3];
            }
            r[i] = f;
        }
    };
    const int64_t ntiles = (T + kSelTile - 1) / kSelTile;
    int64_t tile = blockIdx.x;
    if (tile < ntiles) load(tile);
    for (; tile < ntiles; tile += gridDim.x) {
        const int64_t next = tile + gridDim.x;
        auto store_pass = [&](int, float* sc) {
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int p = tid + kSelThreads * i;
                const int row = p / (BE / 4), c4 = 4 * (p % (BE / 4));
                *reinterpret_cast<float4*>(sc + row * EC::RS + c4) = r[i];
            }
            if (next < ntiles) load(next);
        };
        epi_tile<EC, false>(a, 1, 0, tile * kSelTile, smem, store_pass);
    }
    flush_hist(reinterpret_cast<const int*>(smem + EC::OFF_HIST), a.counts, E);
}

template <int BE>
hipError_t launch_select_be(const RouterArgs& a, const float* scores, hipStream_t stream) {
    const int64_t ntiles = (a.T + kSelTile - 1) / kSelTile;
    int cus = 0;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        cus = 256;
    const int grid = (int)(ntiles < cus ? ntiles : cus);
    hipLaunchKernelGGL((select_kernel<BE>), dim3(grid), dim3(kSelThreads), 0, stream, a, scores);
    return hipGetLastError();
}


// ---------------------------------------------------------------------------
// Register-resident selection.
constexpr int kRegCap = 64;    // candidate list entries per token
constexpr int kRegStage = 4;   // marked chunks per lane staged in LDS

// DPP rotation by R lanes inside each 16-lane row.
template <int R>
__device__ __forceinline__ unsigned row_ror(unsigned x) {
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x120 + R, 0xF, 0xF, false);
}
template <int R>
__device__ __forceinline__ float row_rorf(float x) {
    return __uint_as_float(row_ror<R>(__float_as_uint(x)));
}

// Number of lanes of the row whose value is strictly greater than this lane's.
template <int... R>
__device__ __forceinline__ int row_count_greater(float m, std::integer_sequence<int, R...>) {
    return ((row_rorf<R + 1>(m) > m ? 1 : 0) + ...);
}

// For each of this lane's G values: how many of the row's 16 G values are
// strictly greater.  (The copy is rotated by one lane at a time; unrolled, 3 to
// 4% of a small launch: T = 2048, E = 256, K = 12 9.4 us, 9.7 as a loop.)
template <int G>
__device__ __forceinline__ void row_count_greater(const float (&m)[G], int (&gt)[G]) {
    float o[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        o[g] = m[g];
        gt[g] = 0;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
#pragma unroll
            for (int i = 0; i < G; ++i) gt[i] += o[g] > m[i] ? 1 : 0;
            o[g] = row_rorf<1>(o[g]);
        }
    }
}

__device__ __forceinline__ float row_min(float x) {
    x = fminf(x, row_rorf<8>(x));
    x = fminf(x, row_rorf<4>(x));
    x = fminf(x, row_rorf<2>(x));
    return fminf(x, row_rorf<1>(x));
}

// Row-wide maximum of a 64-bit rank key; every lane of the row gets it.
template <int R>
__device__ __forceinline__ void row_max_key_step(unsigned long long& k) {
    const unsigned lo = row_ror<R>((unsigned)k), hi = row_ror<R>((unsigned)(k >> 32));
    const unsigned long long o = ((unsigned long long)hi << 32) | lo;
    k = o > k ? o : k;
}
__device__ __forceinline__ unsigned long long row_max_key(unsigned long long k) {
    row_max_key_step<8>(k);
    row_max_key_step<4>(k);
    row_max_key_step<2>(k);
    row_max_key_step<1>(k);
    return k;
}

__device__ __forceinline__ float f4_at(const float4& v, int q) {
    return q == 0 ? v.x : q == 1 ? v.y : q == 2 ? v.z : v.w;
}

// Heavy ties (a candidate list that would overflow): K rounds over the row's
// biased scores by the token's 16 lanes (one DPP row, all active).  Round r
// takes the largest rank key strictly below the previous round's pick.  Rank
// keys order (v descending, index ascending) with -0 == +0, and every real
// column's key is above the key 0 a round starts from -- -inf included, so a
// row with fewer than K finite biased scores still picks its -inf columns by
// lowest index.  Each round reads the row again, one float4 at a time (from
// L2), so that this rare path adds few registers to the main path's.
template <int NV>
__device__ __forceinline__ void overflow_select(const float* row, const float* bias_s, unsigned vmask, int j, int K,
                                                int* sel_i, float* sel_s) {
    unsigned long long prev = ~0ull;
    for (int r = 0; r < K; ++r) {
        unsigned long long best = 0ull;
#pragma unroll 1
        for (int c = 0; c < NV; ++c) {
            if ((vmask >> c) & 1u) {
                const int col0 = 4 * (16 * c + j);
                const float4 s4 = *reinterpret_cast<const float4*>(row + col0);
                const float4 b4 = *reinterpret_cast<const float4*>(bias_s + col0);
                const float4 v4 = make_float4(s4.x + b4.x, s4.y + b4.y, s4.z + b4.z, s4.w + b4.w);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const unsigned long long kk = rank_key(f4_at(v4, q), col0 + q);
                    if (kk < prev && kk > best) best = kk;
                }
            }
        }
        best = row_max_key(best);
        prev = best;
        if (j == (r & 15)) {
            const int e = (int)~(unsigned)best;
            sel_i[r] = e;
            sel_s[r] = row[e];
        }
    }
}

// NV: float4 chunks per lane (64 NV >= E).  Lane j of a token's row owns the
// columns 4 (16 c + j) .. +3 for c < NV.  G: group maxima per lane (1, 2 or 4).
// TAIL: the last workgroup applies the controller update.
template <int NV, int WAVES, int G, bool TAIL>
__global__ __launch_bounds__(64 * WAVES) void select_reg_kernel(RouterArgs a, const float* __restrict__ scores,
                                                                CtrlArgs ctrl) {
    constexpr int BE = 64 * NV;
    constexpr int TPB = 4 * WAVES;  // tokens per workgroup tile (4 per wave)
    constexpr int kMaxSel = G == 1 ? 10 : G == 2 ? 16 : kMaxK;  // largest K
    __shared__ __attribute__((aligned(16))) float bias_s[BE];
    __shared__ int hist[BE];
    __shared__ int cnt[TPB];
    // (one entry of padding: the four tokens of a wave read distinct banks)
    __shared__ unsigned long long lkey[TPB][kRegCap + 1];
    __shared__ float lsc[TPB][kRegCap + 1];
    constexpr int SR = G == 1 ? 10 : kMaxSel + 1;  // row stride: the wave's four tokens in distinct banks
    __shared__ int sel_i[TPB][SR];
    __shared__ float sel_s[TPB][SR];
    // each lane's first kRegStage marked chunks, copied from its registers
    // (slot-major, so a wave's copies are consecutive 16-byte units)
    __shared__ float4 staged[kRegStage][64 * WAVES];

    const int tid = threadIdx.x;
    const int E = a.E, K = a.K;
    const int64_t T = a.T;
    for (int i = tid; i < BE; i += blockDim.x) {
        bias_s[i] = i < E ? a.bias[i] : 0.0f;
        hist[i] = 0;
    }
    __syncthreads();

    const int lane = tid & 63;
    const int j = lane & 15;
    const int slot = (tid >> 6) * 4 + (lane >> 4);  // token of the tile
    unsigned vmask = 0;                              // chunks holding real columns
#pragma unroll
    for (int c = 0; c < NV; ++c) vmask |= (4 * (16 * c + j) < E ? 1u : 0u) << c;

    const int64_t ntiles = (T + TPB - 1) / TPB;
    for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int64_t t = tile * TPB + slot;
        const bool valid = t < T;  // uniform over the row
        const float* row = scores + (valid ? t : 0) * (int64_t)E;

        float4 sv[NV];
        // a tile of real tokens whose rows fill all 64 NV columns loads
        // without per-chunk conditions (uniform over the workgroup)
        if (64 * NV == E && (tile + 1) * TPB <= T) {
#pragma unroll
            for (int c = 0; c < NV; ++c) sv[c] = *reinterpret_cast<const float4*>(row + 4 * (16 * c + j));
        } else {
#pragma unroll
            for (int c = 0; c < NV; ++c) {
                sv[c] = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
                if (valid && ((vmask >> c) & 1u)) sv[c] = *reinterpret_cast<const float4*>(row + 4 * (16 * c + j));
            }
        }
        // chunk and lane maxima of v = s + b
        float cm[NV];
        float m[G];
#pragma unroll
        for (int g = 0; g < G; ++g) m[g] = -INFINITY;
#pragma unroll
        for (int c = 0; c < NV; ++c) {
            const float4 b4 = *reinterpret_cast<const float4*>(bias_s + 4 * (16 * c + j));
            const float v0 = sv[c].x + b4.x, v1 = sv[c].y + b4.y, v2 = sv[c].z + b4.z, v3 = sv[c].w + b4.w;
            const float v01 = fmaxf(v0, v1), v23 = fmaxf(v2, v3);
            cm[c] = fmaxf(v01, v23);
            if constexpr (G == 1) {
                m[0] = fmaxf(m[0], cm[c]);
            } else if constexpr (G == 2) {
                m[0] = fmaxf(m[0], v01);
                m[1] = fmaxf(m[1], v23);
            } else {
                m[0] = fmaxf(m[0], v0);
                m[1] = fmaxf(m[1], v1);
                m[2] = fmaxf(m[2], v2);
                m[3] = fmaxf(m[3], v3);
            }
        }
        // tau = the K-th largest of the row's 16 G group maxima: K distinct
        // elements reach it, so every element of the top-K does.  Padding
        // groups (-inf) make tau -inf when fewer than K groups hold real
        // columns.
        int gt[G];
        if constexpr (G == 1) gt[0] = row_count_greater(m[0], std::make_integer_sequence<int, 15>{});
        else row_count_greater<G>(m, gt);
        float low = INFINITY;
#pragma unroll
        for (int g = 0; g < G; ++g) low = fminf(low, gt[g] < K ? m[g] : INFINITY);
        const float tau = row_min(low);

        unsigned cmask = 0;
#pragma unroll
        for (int c = 0; c < NV; ++c) cmask |= (cm[c] >= tau ? 1u : 0u) << c;
        cmask &= valid ? vmask : 0u;

        if (j == 0) cnt[slot] = 0;
        // the first kRegStage marked chunks go from registers to LDS, in
        // ascending chunk order (the order the loop below takes them)
        {
            int k = 0;
#pragma unroll
            for (int c = 0; c < NV; ++c) {
                if ((cmask >> c) & 1u) {
                    if (k < kRegStage) staged[k][tid] = sv[c];
                    ++k;
                }
            }
        }
        wave_sync();
        // candidates: the values >= tau of the marked chunks, appended to the
        // token's list (list order is irrelevant: ranks are counted below);
        // a lane's chunks past the staged ones are read again from memory
        int taken = 0;
        while (__ballot(cmask != 0u) != 0) {
            if (cmask != 0u) {
                const int c = __ffs(cmask) - 1;
                cmask &= cmask - 1u;
                const int col0 = 4 * (16 * c + j);
                const float4 s4 = taken < kRegStage ? staged[taken][tid]
                                                    : *reinterpret_cast<const float4*>(row + col0);
                ++taken;
                const float4 b4 = *reinterpret_cast<const float4*>(bias_s + col0);
                const float4 v4 = make_float4(s4.x + b4.x, s4.y + b4.y, s4.z + b4.z, s4.w + b4.w);
                const int n4 = (v4.x >= tau) + (v4.y >= tau) + (v4.z >= tau) + (v4.w >= tau);
                int p = atomicAdd(&cnt[slot], n4);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (f4_at(v4, q) >= tau) {
                        if (p < kRegCap) {
                            lkey[slot][p] = rank_key(f4_at(v4, q), col0 + q);
                            lsc[slot][p] = f4_at(s4, q);
                        }
                        ++p;
                    }
                }
            }
        }
        wave_sync();

        const int n = cnt[slot];
        const bool over = n > kRegCap;  // uniform over the row
        const int nl = over ? 0 : n;
        int nmax = __builtin_amdgcn_readlane(nl, 0);
        nmax = max(nmax, __builtin_amdgcn_readlane(nl, 16));
        nmax = max(nmax, __builtin_amdgcn_readlane(nl, 32));
        nmax = max(nmax, __builtin_amdgcn_readlane(nl, 48));
        // rank of each listed candidate = the number of list keys above it;
        // the lanes take the entries in groups of 16.  The lists of the wave's
        // tokens are filled up to a common length with key 0, below every key,
        // so the sweep needs no test per key and token.
        const int nfull = (nmax + 3) & ~3;  // <= kRegCap
        for (int e = nl + j; e < nfull; e += 16) lkey[slot][e] = 0ull;
        wave_sync();
        for (int base = 0; base < nmax; base += 16) {
            const int me = base + j;
            const unsigned long long km = me < nl ? lkey[slot][me] : 0ull;
            int rk = 0;
            for (int e = 0; e < nfull; e += 4) {
                const unsigned long long q0 = lkey[slot][e], q1 = lkey[slot][e + 1];
                const unsigned long long q2 = lkey[slot][e + 2], q3 = lkey[slot][e + 3];
                rk += (q0 > km ? 1 : 0) + (q1 > km ? 1 : 0) + (q2 > km ? 1 : 0) + (q3 > km ? 1 : 0);
            }
            if (me < nl && rk < K) {
                sel_i[slot][rk] = (int)~(unsigned)km;
                sel_s[slot][rk] = lsc[slot][me];
            }
        }

        if (over) {
            overflow_select<NV>(row, bias_s, vmask, j, K, &sel_i[slot][0], &sel_s[slot][0]);
        }
        wave_sync();

        if (valid && j < K) {
            // den: fp32 sum of the selected unbiased scores in rank order
            float den = 0.0f;
            for (int r = 0; r < K; ++r) den = den + sel_s[slot][r];
#pragma unroll
            for (int r = j; r < kMaxSel; r += 16) {
                if (r < K) {
                    const int idx = sel_i[slot][r];
                    a.idx[t * K + r] = idx;
                    a.w[t * K + r] = (den == 0.0f) ? 1.0f / (float)K : sel_s[slot][r] / den;
                    atomicAdd(&hist[idx], 1);
                }
            }
        }
        wave_sync();
    }
    __syncthreads();
    flush_hist(hist, a.counts, E);
    if constexpr (TAIL) {
        __shared__ CtrlScratch csh;
        controller_tail<1024 / (64 * WAVES)>(a.counts, E, ctrl.Ki, ctrl.Kd, ctrl.sign_mode, ctrl.center, ctrl.bias,
                                             ctrl.e_prev, ctrl.step, ctrl.status, ctrl.stats, ctrl.ticket, csh);
    }
}

// Workgroup shape.  Every workgroup flushes its histogram with one device
// atomic per non-zero bin, so fewer, larger workgroups issue fewer atomics to
// the same few counters; small batches leave CUs idle that way and take 8 waves,
// the longer the rows and the larger K (the more work per token) the longer.  us
// for 4, 8 and 16 waves: E = 96, K = 4: T = 1536 8.4, 7.5, 7.6, T = 4096 12.2, 9.3, 8.4;
// E = 256, K = 4: T = 2048 9.1, 7.9, 8.0, T = 4096 11.8, 9.3, 8.6; E = 512, K = 4: T = 4096
// 11.5, 9.7, 9.5, K = 8 12.8, 10.4, 10.4; E = 1024, K = 4: T = 2560 10.4, 10.0, 11.7, T =
// 4096 11.9, 11.0, 12.0; E = 256, K = 16: T = 4096 14.5, 11.7, 12.1; E = 32, K = 32: T =
// 8192 -, 12.4, 13.7.  Batches of several 4-wave workgroups, but few, gain up to 5%
// on those (E = 1024, K = 20: T = 64 13.6, 14.0, 14.0), unless the last workgroup's
// controller update, which has more threads in a larger one, weighs more (router
// step, K <= 10, T = 32: 8 waves 0.94 of the time of 4).
constexpr int kRegWaves = 16;
template <int NV, int G>
constexpr int64_t kRegFewTokens = G > 1 ? 2048 * G : NV >= 8 ? 4096 : 2048;  // up to here 8 waves
constexpr int64_t kRegOneTokens = 16, kRegTinyTokens = 256;  // above and up to these 4 waves

template <int NV, int WAVES, int G>
hipError_t launch_select_waves(const RouterArgs& a, const float* scores, const CtrlArgs& ctrl, int cus,
                               hipStream_t stream) {
    constexpr int TPB = 4 * WAVES;
    const int64_t ntiles = (a.T + TPB - 1) / TPB;
    // one round of workgroups over the CUs; more tiles are walked grid-stride
    const int64_t cap = (int64_t)cus * (kRegWaves / WAVES);
    const int grid = (int)(ntiles < cap ? ntiles : cap);
    if (ctrl.ticket)
        hipLaunchKernelGGL((select_reg_kernel<NV, WAVES, G, true>), dim3(grid), dim3(64 * WAVES), 0, stream, a, scores,
                           ctrl);
    else
        hipLaunchKernelGGL((select_reg_kernel<NV, WAVES, G, false>), dim3(grid), dim3(64 * WAVES), 0, stream, a,
                           scores, ctrl);
    return hipGetLastError();
}

template <int NV, int G>
hipError_t launch_select_reg(const RouterArgs& a, const float* scores, const CtrlArgs& ctrl, hipStream_t stream) {
    int cus = 0;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        cus = 256;
    if (a.T > kRegOneTokens && a.T <= kRegTinyTokens && (G == 4 || !ctrl.ticket))
        return launch_select_waves<NV, 4, G>(a, scores, ctrl, cus, stream);
    if (a.T <= kRegFewTokens<NV, G>) return launch_select_waves<NV, 8, G>(a, scores, ctrl, cus, stream);
    // the widest rows with several group maxima need more than the 128 VGPRs of
    // a 16-wave workgroup
    constexpr int waves = (NV >= 16 && G >= 2) || (NV >= 12 && G == 4) ? kRegWaves / 2 : kRegWaves;
    return launch_select_waves<NV, waves, G>(a, scores, ctrl, cus, stream);
}

template <int G>
hipError_t launch_select_groups(const RouterArgs& a, const float* scores, const CtrlArgs& ctrl, hipStream_t stream) {
    if (a.E <= 64) return launch_select_reg<1, G>(a, scores, ctrl, stream);
    if (a.E <= 128) return launch_select_reg<2, G>(a, scores, ctrl, stream);
    if (a.E <= 256) return launch_select_reg<4, G>(a, scores, ctrl, stream);
    if (a.E <= 512) return launch_select_reg<8, G>(a, scores, ctrl, stream);
    if (a.E <= 768) return launch_select_reg<12, G>(a, scores, ctrl, stream);
    return launch_select_reg<16, G>(a, scores, ctrl, stream);
}

}  // namespace

hipError_t launch_fill_i32(int32_t* p, int32_t value, int64_t n, hipStream_t stream) {
    int64_t blocks = (n + 255) / 256;
    if (blocks > 1024) blocks = 1024;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(fill_i32_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, p, value, n);
    return hipGetLastError();
}

hipError_t launch_select_step(const RouterArgs& a, const float* scores, const CtrlArgs* ctrl, hipStream_t stream) {
    CtrlArgs c{};
    if (ctrl) c = *ctrl;
    if (a.K <= 10) return launch_select_groups<1>(a, scores, c, stream);
    if (a.K <= 16) return launch_select_groups<2>(a, scores, c, stream);
    return launch_select_groups<4>(a, scores, c, stream);
}

hipError_t launch_select_from_scores(const float* scores, const float* bias, int64_t T, int E, int K, int32_t* idx,
                                     float* w, int32_t* counts, hipStream_t stream) {
    RouterArgs a{};
    a.bias = bias;
    a.T = T;
    a.E = E;
    a.K = K;
    a.idx = idx;
    a.w = w;
    a.counts = counts;
    // 16-byte pieces need aligned rows
    if (E % 4 == 0 && (reinterpret_cast<uintptr_t>(scores) & 15) == 0)
        return launch_select_step(a, scores, nullptr, stream);
    if (E <= 256) return launch_select_be<256>(a, scores, stream);
    if (E <= 512) return launch_select_be<512>(a, scores, stream);
    if (E <= 768) return launch_select_be<768>(a, scores, stream);
    return launch_select_be<1024>(a, scores, stream);
}

}  // namespace idb
