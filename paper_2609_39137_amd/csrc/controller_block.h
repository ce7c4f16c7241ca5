// The ID bias controller update (Algorithm 1, Eq. rapid-update), the load
// statistics (Eq. vio) and the update's diagnostics as a device function of
// one workgroup: the stand-alone controller kernel, the batched kernel of many
// layers (a workgroup each) and the router tail that runs it after the last
// workgroup of the slice merge or of the selection.
//
// O(E) work on at most 1024 experts, so bound by latency: memory round trips,
// barriers and the steps of the reductions.  Integers are reduced by DPP row
// rotations and scalar reads (a ds_bpermute shuffle costs an LDS round trip
// per step), the waves' partials by one LDS read and a row rotation each.
#pragma once

#include "common.h"

namespace idb {

// LDS scratch of controller_block.
struct CtrlScratch {
    int part[2][4][16];  // per-wave partials of the workgroup reductions (two banks, alternating)
    float tree[1024];
    float root;
};

// LDS scratch of the diagnostics (controller_block with a diag pointer).
struct DiagScratch {
    int wcnt[2][3][16];  // per-wave counts of the threshold search (two banks, alternating)
    double tree[1024];
};

// Leaves of the centering tree: the next power of two >= E.
__host__ __device__ inline int ctrl_tree_size(int E) {
    int P = 1;
    while (P < E) P <<= 1;
    return P;
}

struct AddOp {
    __device__ __forceinline__ int operator()(int a, int b) const { return a + b; }
};
struct MaxOp {
    __device__ __forceinline__ int operator()(int a, int b) const { return max(a, b); }
};
struct MinOp {
    __device__ __forceinline__ int operator()(int a, int b) const { return min(a, b); }
};

// Reduction over a 16-lane row (every lane of it gets the result; all active).
template <class Op>
__device__ __forceinline__ int row_reduce(int v, Op op) {
    v = op(v, row_rot<8>(v));
    v = op(v, row_rot<4>(v));
    v = op(v, row_rot<2>(v));
    return op(v, row_rot<1>(v));
}
// Reduction over the wave (uniform result).
template <class Op>
__device__ __forceinline__ int wave_reduce(int v, Op op) {
    v = row_reduce(v, op);
    return op(op(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
              op(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

// A sum of int32 values in 64 bits as two 32-bit sums: of the low halfwords
// and of the (signed) high ones; exact for up to 32768 values.
struct SplitSum {
    int lo = 0, hi = 0;
    __device__ __forceinline__ void add(int n) {
        lo += n & 0xffff;
        hi += n >> 16;
    }
};
__device__ __forceinline__ long long split_total(int lo, int hi) { return (long long)hi * 65536 + lo; }

// The fixed pairwise tree over P leaves, leaf i0 + q nt in v[q] of thread i0:
// level h adds leaf j + h into leaf j for j < h, h = P/2, ..., 1.  Levels
// h >= nt pair two leaves of one thread; levels nt/2 .. 64 pair the same lane
// of two waves (through mem; wave 0 adds them in registers); the last six run
// inside wave 0 (lane moves that add the same pairs).  Wave 0's lanes return
// the root.  One barrier when more than one wave holds leaves.  kOneWave: the
// workgroup is one wave (mem unused).
template <bool kOneWave, int kPer, class V>
__device__ inline V block_tree_sum(V (&v)[kPer], int P, V* mem) {
    const int i0 = threadIdx.x, nt = kOneWave ? 64 : blockDim.x, lane = i0 & 63, wv = kOneWave ? 0 : i0 >> 6;
#pragma unroll
    for (int d = kPer / 2; d >= 1; d >>= 1)
        if (2 * d * nt <= P)
#pragma unroll
            for (int q = 0; q < d; ++q) v[q] = v[q] + v[q + d];
    const int NP = P < nt ? P : nt;  // tree nodes left, node i0 in thread i0
    V a = v[0];
    if (!kOneWave && NP > 64) {
        if (i0 >= 64 && i0 < NP) mem[i0] = a;
        __syncthreads();
        if (wv == 0) {
            V r[16];  // node 64 w + lane, w < NP / 64 <= 16
            r[0] = a;
#pragma unroll
            for (int w = 1; w < 16; ++w) r[w] = (w < NP / 64) ? mem[64 * w + lane] : (V)0;
#pragma unroll
            for (int hw = 8; hw >= 1; hw >>= 1)
                if (hw < NP / 64)
#pragma unroll
                    for (int w = 0; w < hw; ++w) r[w] = r[w] + r[w + hw];
            a = r[0];
        }
    }
    if (wv == 0) {
        if (NP > 32) a = a + __shfl_xor(a, 32);
        if (NP > 16) a = a + __shfl_xor(a, 16);
        if (NP >= 16) {
            // a rotation by half the period: every lane ends with the root
            a = a + row_rot<8>(a);
            a = a + row_rot<4>(a);
            a = a + row_rot<2>(a);
            a = a + row_rot<1>(a);
        } else {
            for (int h = NP >> 1; h >= 1; h >>= 1) {
                const V up = __shfl_down(a, h);
                if (lane < h) a = a + up;
            }
            a = __shfl(a, 0);
        }
    }
    return a;
}

// The thread's experts' bias and previous error (experts i0, i0 + nt, ...).
template <int kPer>
__device__ __forceinline__ void controller_load_state(const float* __restrict__ bias,
                                                      const float* __restrict__ e_prev, int E, float (&b0)[kPer],
                                                      float (&ep0)[kPer]) {
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int i = threadIdx.x + q * blockDim.x;
        b0[q] = (i < E) ? bias[i] : 0.0f;
        ep0[q] = (i < E) ? e_prev[i] : 0.0f;
    }
}

// The whole O(E) update on one workgroup whose size is a multiple of 64, each
// thread taking experts i, i + blockDim, ... (kPer of them): needs
// kPer * blockDim >= P, the centering tree's size, and E <= 1024.  b0, ep0: the
// state (controller_load_state).  With a non-null stats pointer it also writes
// MaxVio/MinVio of the same counts; with a non-null diag pointer (and dsh), the
// update's diagnostics: diag[0] the active-gate fraction #{g_i = 1}/E, diag[1]
// the share of the assignments on the m = ceil(E/10) busiest experts (the sum
// of the m largest counts over S), diag[2] the inactive-expert ratio
// #{n_i = 0}/E, diag[3] the mean |b_new - b_old| summed in fp64 over the same
// pairwise tree; NaN x 4 when the update does not run.
// Reductions: exact integer sums/extrema (order-free); the centering mean with
// the fixed pairwise tree of block_tree_sum, P = next power of two >= E.
// kOneWave: the workgroup is one wave, which needs no LDS and no barrier (sh and
// dsh unused).
template <int kPer, bool kCoherentCounts = false, bool kOneWave = false>
__device__ inline void controller_block(const int32_t* __restrict__ counts, int E, int P, float Ki, float Kd,
                                        int sign_mode, int center, const float (&b0)[kPer], const float (&ep0)[kPer],
                                        float* __restrict__ bias, float* __restrict__ e_prev,
                                        int64_t* __restrict__ step, int32_t* __restrict__ status,
                                        double* __restrict__ stats, CtrlScratch& sh, double* __restrict__ diag = nullptr,
                                        DiagScratch* dsh = nullptr) {
#pragma clang fp contract(off)
    const int i0 = threadIdx.x, nt = kOneWave ? 64 : blockDim.x;
    const int lane = i0 & 63, wv = kOneWave ? 0 : i0 >> 6, nw = nt >> 6;
    int n[kPer];
    SplitSum sum;
    int mx = INT32_MIN, mn = INT32_MAX;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int i = i0 + q * nt;
        // counts written by atomics of other workgroups of the same launch
        // are read with agent-scope loads.
        n[q] = (i >= E) ? 0
               : kCoherentCounts ? __hip_atomic_load(counts + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                 : counts[i];
        if (i < E) {
            sum.add(n[q]);
            mx = max(mx, n[q]);
            mn = min(mn, n[q]);
        }
    }
    // each wave's four integers to LDS; every row then reduces the waves' partials
    int red[4] = {wave_reduce(sum.lo, AddOp{}), wave_reduce(sum.hi, AddOp{}), wave_reduce(mx, MaxOp{}),
                  wave_reduce(mn, MinOp{})};
    const int pw = lane & 15;
    const bool has = pw < nw;
    if constexpr (!kOneWave) {
        if (lane == 0)
#pragma unroll
            for (int c = 0; c < 4; ++c) sh.part[0][c][wv] = red[c];
        __syncthreads();
        red[0] = row_reduce(has ? sh.part[0][0][pw] : 0, AddOp{});
        red[1] = row_reduce(has ? sh.part[0][1][pw] : 0, AddOp{});
        red[2] = row_reduce(has ? sh.part[0][2][pw] : INT32_MIN, MaxOp{});
        red[3] = row_reduce(has ? sh.part[0][3][pw] : INT32_MAX, MinOp{});
    }
    // Total assignments S = E * nbar (Eq. pid-error).
    const long long S = split_total(red[0], red[1]);
    mx = red[2];
    mn = red[3];
    if (stats && i0 == nt - 1) {
        // MaxVio, MinVio (Eq. vio): one fp64 division of an exact integer
        // numerator each; NaN for an empty batch.  (The last wave: wave 0
        // has the centering tree's serial part.)
        if (S == 0) {
            stats[0] = __builtin_nan("");
            stats[1] = __builtin_nan("");
        } else {
            stats[0] = (double)((long long)E * mx - S) / (double)S;
            stats[1] = (double)(S - (long long)E * mn) / (double)S;
        }
    }
    if (mn < 0 || S == 0) {
        // Invalid or empty batch: report it and leave the state untouched.
        if (i0 == 0) {
            *status = mn < 0 ? kStatusInvalid : kStatusEmpty;
            if (diag)
                for (int q = 0; q < 4; ++q) diag[q] = __builtin_nan("");
        }
        return;
    }
    float e[kPer], b[kPer];
    int gates = 0;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int i = i0 + q * nt;
        e[q] = 0.0f;
        b[q] = 0.0f;
        if (i < E) {
            // Normalised load error e = (nbar - n)/nbar = (S - E n)/S: exact
            // integer numerator, one correctly rounded fp64 division, then fp32.
            const long long num = S - (long long)E * (long long)n[q];
            e[q] = (float)((double)num / (double)S);
            const float ep = ep0[q];
            const float de = e[q] - ep;  // Eq. rapid-delta
            // Worsening gate (Eq. rapid-gate) as a sign test: open iff the
            // previous error and its change are both positive or both negative.
            const bool g = (ep > 0.0f && de > 0.0f) || (ep < 0.0f && de < 0.0f);
            float u;
            if (sign_mode) {
                const float sg = (e[q] > 0.0f) ? 1.0f : ((e[q] < 0.0f) ? -1.0f : 0.0f);
                u = Ki * sg;  // DeepSeek fixed-step integral
            } else {
                u = Ki * e[q];  // magnitude-aware integral
            }
            b[q] = b0[q] + u;
            if (g) {
                const float dterm = Kd * de;  // gated, accumulated derivative
                b[q] = b[q] + dterm;
            }
            gates += g ? 1 : 0;
        }
    }
    // Zero-mean centering (second line of Eq. rapid-update)
    float m = 0.0f;
    if (center) {
        float v[kPer];
#pragma unroll
        for (int q = 0; q < kPer; ++q) v[q] = (i0 + q * nt < E) ? b[q] : 0.0f;
        if constexpr (kOneWave) {
            const float a = block_tree_sum<true>(v, P, (float*)nullptr);
            m = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, a))) / (float)E;
        } else {
            const float a = block_tree_sum<false>(v, P, sh.tree);
            if (i0 == 0) sh.root = a;
            __syncthreads();
            m = sh.root / (float)E;
        }
    }
    float nb[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int i = i0 + q * nt;
        nb[q] = center ? (b[q] - m) : b[q];
        if (i < E) {
            bias[i] = nb[q];
            e_prev[i] = e[q];
        }
    }
    if (i0 == 0) {
        *step = *step + 1;
        *status = kStatusOk;
    }
    if (!diag) return;
    // diagnostics of this update
    int zeros = 0;
    double d[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const bool real = i0 + q * nt < E;
        zeros += (real && n[q] == 0) ? 1 : 0;
        d[q] = real ? (double)fabsf(nb[q] - b0[q]) : 0.0;
    }
    // The m = ceil(E/10) largest counts: their sum does not depend on how ties
    // are ranked, so it is sum(n_i > th) + (m - #{n_i > th}) th with th the
    // m-th largest count, the largest v with #{n_i >= v} >= m, found from the
    // top (counts are >= 0 here, mx the largest): two bits at a time where a step
    // costs a barrier, one at a time (fewer ballots) in one wave.
    const int mtop = (E + 9) / 10;
    int th = 0;
    constexpr int kBits = kOneWave ? 1 : 2, kTries = (1 << kBits) - 1;
    const int top = (31 - __builtin_clz((unsigned)mx | 1u)) / kBits * kBits;  // the lowest of the highest bits
    for (int bit = top, bank = 0; bit >= 0; bit -= kBits, bank ^= 1) {
        int c[kTries] = {};
#pragma unroll
        for (int q = 0; q < kPer; ++q)
#pragma unroll
            for (int t = 0; t < kTries; ++t)
                c[t] += __builtin_popcountll(__builtin_amdgcn_ballot_w64(
                    i0 + q * nt < E && (unsigned)n[q] >= ((unsigned)th | ((unsigned)(t + 1) << bit))));
        if constexpr (!kOneWave) {
            if (lane == 0)
#pragma unroll
                for (int t = 0; t < kTries; ++t) dsh->wcnt[bank][t][wv] = c[t];
            __syncthreads();  // the other bank was last read before the previous barrier
#pragma unroll
            for (int t = 0; t < kTries; ++t) c[t] = row_reduce(has ? dsh->wcnt[bank][t][pw] : 0, AddOp{});
        }
        int add = 0;
#pragma unroll
        for (int t = 0; t < kTries; ++t) add += c[t] >= mtop ? 1 : 0;
        th = (int)((unsigned)th | ((unsigned)add << bit));
    }
    SplitSum above;
    int nabove = 0;
#pragma unroll
    for (int q = 0; q < kPer; ++q)
        if (i0 + q * nt < E && n[q] > th) {
            above.add(n[q]);
            nabove += 1;
        }
    const int packed = gates << 16 | zeros;  // at most 1024 each
    int dred[4] = {wave_reduce(above.lo, AddOp{}), wave_reduce(above.hi, AddOp{}), wave_reduce(nabove, AddOp{}),
                   wave_reduce(packed, AddOp{})};
    double drift;
    if constexpr (kOneWave) {
        drift = block_tree_sum<true>(d, P, (double*)nullptr);
    } else {
        if (lane == 0)
#pragma unroll
            for (int c = 0; c < 4; ++c) sh.part[1][c][wv] = dred[c];
        drift = block_tree_sum<false>(d, P, dsh->tree);
        __syncthreads();
#pragma unroll
        for (int c = 0; c < 4; ++c) dred[c] = row_reduce(has ? sh.part[1][c][pw] : 0, AddOp{});
    }
    if (wv == 0) {
        const long long sum_above = split_total(dred[0], dred[1]);
        const int na = dred[2], gz = dred[3];
        if (lane == 0) {
            const long long TOP = sum_above + (long long)(mtop - na) * (long long)th;
            diag[0] = (double)(gz >> 16) / (double)E;
            diag[1] = (double)TOP / (double)S;
            diag[2] = (double)(gz & 0xffff) / (double)E;
            diag[3] = drift / (double)E;
        }
    }
}

// Run by every thread of each workgroup of a launch once it is done with
// counts: the workgroup that finishes last (ticket) runs controller_block on
// the complete counts.  The counts are written only by agent-scope atomics
// (performed at the device's coherence point) and read only by agent-scope
// loads (served there too), so no cache write-back or invalidation is needed:
// every wave waits for its own memory operations (the count atomics) to
// complete, the barrier collects the workgroup, and one thread takes the
// ticket; the last workgroup reads the counts after its ticket returns.  The
// controller state it reads is written by no other workgroup of the launch.
template <int kPer>
__device__ inline void controller_tail(const int32_t* counts, int E, float Ki, float Kd, int sign_mode, int center,
                                       float* bias, float* e_prev, int64_t* step, int32_t* status, double* stats,
                                       unsigned* ticket, CtrlScratch& sh) {
    __shared__ int last;
    // the state is written by no other workgroup of the launch: its loads run
    // under the wait for the ticket (a memory round trip less for the last one)
    float b0[kPer], ep0[kPer];
    controller_load_state(bias, e_prev, E, b0, ep0);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0)
        last = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
    __syncthreads();
    if (!last) return;
    controller_block<kPer, true>(counts, E, ctrl_tree_size(E), Ki, Kd, sign_mode, center, b0, ep0, bias, e_prev, step,
                                 status, stats, sh);
}

}  // namespace idb
