// Routing entropies (Sec. 4.3), averaged over the tokens of a batch:
//   H_topK = -sum_r w_r log w_r over a token's gate weights (0 log 0 = 0),
//            natural logarithms in fp64;
//   H_full = -sum_e p_e log p_e, p_e = c_e / C, c_e = max(fl32(s_e + b_e), 0),
//            C = sum_e c_e, evaluated as log C - ln 2 (sum_e c_e log2 c_e) / C
//            (H_full = 0 when C = 0), each c_e log2 c_e with the hardware
//            fp32 log2 and summed in fp64 (below the smallest normal fp32 c_e
//            keeps its value and takes that number's logarithm).
// The softmax form (the auxiliary-loss router, whose selection scores are the
// softmax probabilities of its logits): H_full = log Z - (sum_e t_e (z_e - M))
// / Z with M the token's largest logit, t_e = exp(z_e - M) from the hardware
// exp2 in fp32 and Z = sum_e t_e, both sums in fp64.
// Deterministic: a fixed grid of kEntropyBlocks workgroups with fixed token
// assignments and fixed reduction trees writes per-workgroup partial sums,
// which one wave adds in a fixed order.
#include "common.h"
#include "internal.h"

#pragma clang fp contract(off)

namespace idb {

namespace {

constexpr int kEntAhead = 2;  // rows a wave has in flight
// Up to this many tokens a workgroup has 256 threads, else 512: fewer waves to
// start and to reduce over when most have no token or one.  us, 256 / 512 threads:
// softmax, K = 1: T = 200, E = 1024 6.8 / 7.7; T = 4096, E = 256 7.2 / 8.2; T = 8192, E =
// 256 8.8 / 9.3; T = 16384, E = 512 13.6 / 13.3, E = 404 14.7 / 13.9; T = 65536, E = 768
// 44.6 / 39.7.
constexpr int64_t kEntFewTokens = 8192;

template <int NT>
__device__ inline double block_sum_fixed(double v, double* red) {
    // fixed butterfly inside each wave, then the waves in order
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) red[wv] = v;
    __syncthreads();
    double t = 0.0;
    for (int w = 0; w < NT / 64; ++w) t += red[w];
    __syncthreads();
    return t;
}

// A row's values of this lane: columns 4 (lane + 64 p) .. + 3 for p < NP
// (256 NP >= E); `pad` past the row.
template <int NP>
__device__ __forceinline__ void load_row(const float* __restrict__ row, int E, float pad, float (&v)[4 * NP]) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int c0 = 4 * (lane + 64 * p);
        if (c0 + 4 <= E) {
            const f4u f = *reinterpret_cast<const f4u*>(row + c0);
#pragma unroll
            for (int c = 0; c < 4; ++c) v[4 * p + c] = f.v[c];
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) v[4 * p + c] = c0 + c < E ? row[c0 + c] : pad;
        }
    }
}

// Sum over the wave in a fixed order, in every lane: row rotations (which
// cost no LDS round trip), then two exchanges between the rows.
__device__ __forceinline__ double wave_sum(double v) {
    v += row_rot<8>(v);
    v += row_rot<4>(v);
    v += row_rot<2>(v);
    v += row_rot<1>(v);
    v += __shfl_xor(v, 16);
    return v + __shfl_xor(v, 32);
}

// One token's sums Z = sum exp(z - M) and D = sum exp(z - M) (z - M) over its
// logits z (one wave; padding -inf), in every lane.
template <int N>
__device__ __forceinline__ void softmax_sums_wave(const float (&z)[N], double& Z, double& D) {
    float m = -INFINITY;
#pragma unroll
    for (int j = 0; j < N; ++j) m = fmaxf(m, z[j]);
    m = fmaxf(m, row_rot<8>(m));
    m = fmaxf(m, row_rot<4>(m));
    m = fmaxf(m, row_rot<2>(m));
    m = fmaxf(m, row_rot<1>(m));
    m = fmaxf(m, __shfl_xor(m, 16));
    m = fmaxf(m, __shfl_xor(m, 32));
    Z = 0.0;
    D = 0.0;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        if (z[j] != -INFINITY) {
            const float x = z[j] - m;
            const float t = __builtin_amdgcn_exp2f(x * 1.4426950408889634f);
            Z += (double)t;
            D = __builtin_fma((double)t, (double)x, D);
        }
    }
    Z = wave_sum(Z);
    D = wave_sum(D);
}

// One token's sums C = sum c and D = sum c log2 c over its clamped biased
// scores (one wave; padding scores are 0 with bias 0), in every lane.  The
// logarithm of a c below the smallest normal fp32 is that number's (such a term
// is below 2^-119 in size; 0 for c = 0).
template <int N>
__device__ __forceinline__ void clamped_sums_wave(const float (&s)[N], const float (&b)[N], double& C, double& D) {
    C = 0.0;
    D = 0.0;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const float c = fmaxf(s[j] + b[j], 0.0f);
        const double c64 = (double)c;
        C += c64;
        D = __builtin_fma(c64, (double)__builtin_amdgcn_logf(fmaxf(c, 1.17549435e-38f)), D);
    }
    C = wave_sum(C);
    D = wave_sum(D);
}

// H_full of a token from its sums (see the head of the file).
template <bool SOFTMAX>
__device__ inline double entropy_of(double C, double D) {
    constexpr double kLn2 = 0.69314718055994530942;
    if (SOFTMAX) return log(C) - D / C;
    return C > 0.0 ? log(C) - kLn2 * D / C : 0.0;
}

// Bound by the VALU (about 21 instructions per 64 scores, half of them fp64)
// under the read of the scores.  A wave takes every (grid waves)-th token and
// has two rows in flight (four: 22.3 us); only the pieces a row fills are
// computed (NP), and the H_topK terms are spread one per thread over the
// block's run of tokens.  At T = 16384, E = 768, K = 10: 14.4 us (3.5 TB/s;
// 18.0 us with a logarithm and a division per token in every lane, one row
// ahead and two shuffles per reduction step).
template <bool SOFTMAX, int NP, int NT>
__global__ __launch_bounds__(NT) void entropy_partial_kernel(const float* __restrict__ w, int64_t T, int K,
                                                                      const float* __restrict__ scores,
                                                                      const float* __restrict__ bias, int E,
                                                                      double* __restrict__ partial) {
    constexpr int NW = NT / 64;
    __shared__ double red[NW];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t first = (int64_t)blockIdx.x * NW + wv;
    // (from the launch, not the constant: with that the row loads' offsets fold
    // otherwise and E = 768, T = 16384 takes 15.9 us, not 15.2)
    const int64_t step = (int64_t)gridDim.x * NW;
    constexpr float kPad = SOFTMAX ? -INFINITY : 0.0f;
    float buf[kEntAhead][4 * NP], b[4 * NP];
    if (scores) {
#pragma unroll
        for (int k = 0; k < kEntAhead; ++k)
            if (first + k * step < T) load_row<NP>(scores + (first + k * step) * E, E, kPad, buf[k]);
        if constexpr (!SOFTMAX) load_row<NP>(bias, E, 0.0f, b);
    }
    // H_topK: terms of the block's tokens (0 log 0 = 0)
    const int64_t t_lo = T * blockIdx.x / kEntropyBlocks, t_hi = T * (blockIdx.x + 1) / kEntropyBlocks;
    double htop = 0.0;
    for (int64_t i = t_lo * K + tid; i < t_hi * K; i += NT) {
        const double x = (double)w[i];
        if (x > 0.0) htop -= x * log(x);
    }
    // H_full
    double hfull = 0.0, myC = 0.0, myD = 0.0;
    int held = 0;
    if (scores) {
        for (int64_t t0 = first; t0 < T; t0 += kEntAhead * step) {
#pragma unroll
            for (int k = 0; k < kEntAhead; ++k) {
                const int64_t t = t0 + k * step;
                if (t < T) {
                    double C, D;
                    if constexpr (SOFTMAX) softmax_sums_wave(buf[k], C, D);
                    else clamped_sums_wave(buf[k], b, C, D);
                    // lane i keeps the i-th token's sums: the fp64 logarithm
                    // and division are evaluated once per 64 tokens
                    if (lane == held) {
                        myC = C;
                        myD = D;
                    }
                    if (++held == 64) {
                        hfull += entropy_of<SOFTMAX>(myC, myD);
                        held = 0;
                    }
                    if (t + kEntAhead * step < T) load_row<NP>(scores + (t + kEntAhead * step) * E, E, kPad, buf[k]);
                }
            }
        }
        if (lane < held) hfull += entropy_of<SOFTMAX>(myC, myD);
    }
    const double stop = block_sum_fixed<NT>(htop, red);
    const double sfull = block_sum_fixed<NT>(hfull, red);
    if (tid == 0) {
        partial[2 * blockIdx.x] = stop;
        partial[2 * blockIdx.x + 1] = sfull;
    }
}

// One wave: lane l adds the partials l, l + 64, ... in order, then a fixed
// butterfly over the lanes.
__global__ __launch_bounds__(64) void entropy_final_kernel(const double* __restrict__ partial, int nblk, int64_t T,
                                                          int has_scores, double* __restrict__ out) {
    const int lane = threadIdx.x;
    double a = 0.0, b = 0.0;
#pragma unroll 8
    for (int i = lane; i < nblk; i += 64) {
        a += partial[2 * i];
        b += partial[2 * i + 1];
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        a += __shfl_xor(a, o);
        b += __shfl_xor(b, o);
    }
    if (lane == 0) {
        out[0] = a / (double)T;
        out[1] = has_scores ? b / (double)T : __builtin_nan("");
    }
}

template <bool SOFTMAX, int NP>
void launch_partial(const float* gate_w, int64_t T, int K, const float* scores, const float* bias, int E,
                    double* partial, hipStream_t stream) {
    if (T <= kEntFewTokens)
        hipLaunchKernelGGL((entropy_partial_kernel<SOFTMAX, NP, 256>), dim3(kEntropyBlocks), dim3(256), 0, stream,
                           gate_w, T, K, scores, bias, E, partial);
    else
        hipLaunchKernelGGL((entropy_partial_kernel<SOFTMAX, NP, 512>), dim3(kEntropyBlocks), dim3(512), 0, stream,
                           gate_w, T, K, scores, bias, E, partial);
}

}  // namespace

hipError_t launch_routing_entropy(const float* gate_w, int64_t T, int K, const float* scores, const float* bias,
                                  int E, int softmax, double* partial, double* out, hipStream_t stream) {
    const int np = (E + 255) / 256;  // 0 (no scores) to 4
    if (softmax) {
        if (np <= 1) launch_partial<true, 1>(gate_w, T, K, scores, bias, E, partial, stream);
        else if (np == 2) launch_partial<true, 2>(gate_w, T, K, scores, bias, E, partial, stream);
        else if (np == 3) launch_partial<true, 3>(gate_w, T, K, scores, bias, E, partial, stream);
        else launch_partial<true, 4>(gate_w, T, K, scores, bias, E, partial, stream);
    } else {
        if (np <= 1) launch_partial<false, 1>(gate_w, T, K, scores, bias, E, partial, stream);
        else if (np == 2) launch_partial<false, 2>(gate_w, T, K, scores, bias, E, partial, stream);
        else if (np == 3) launch_partial<false, 3>(gate_w, T, K, scores, bias, E, partial, stream);
        else launch_partial<false, 4>(gate_w, T, K, scores, bias, E, partial, stream);
    }
    hipLaunchKernelGGL(entropy_final_kernel, dim3(1), dim3(64), 0, stream, partial, kEntropyBlocks, T,
                       scores ? 1 : 0, out);
    return hipGetLastError();
}

}  // namespace idb
