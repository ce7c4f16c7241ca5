// Quantile Balancing's bias update (Eq. pid-quantile, Eq. pid-quantile-def),
// with the EMA variant the paper uses as a diagnostic: for each expert j,
//   d_ij = fl32(s_ij - alpha_i)                   (margins, -0 read as +0)
//   q_j  = quantile_{1-K/E}(d_.j) = the k-th smallest margin,
//          k = ceil(T (E - K) / E)                (inverted empirical CDF)
//   b_j  = -q_j, or fl32(fl32(rho b_j) + fl32(fl32(1 - rho) (-q_j))) for rho > 0.
// s comes expert-major ([E][T], written by the router in its Quantile
// Balancing mode) and alpha [T] is each token's (K+1)-th largest biased score.
//
// One workgroup per expert finds the exact k-th smallest margin over the
// margins' order-preserving 32-bit keys.  Up to 65536 tokens each thread keeps
// its keys in registers (R <= 64 of them, 512 or 1024 threads; one read of the
// row at any 4-byte alignment) and a sampled bracket narrows them to a short
// list (qb_update_reg_kernel).  Measured at T = 16384, E = 768, K = 10: 19.4 us
// (2.6 TB/s), 19.2 us once the biases have drifted off together (21.4 and 23.6
// us with a threshold from the per-thread maxima, which also needed a full radix
// select from r = T K / E > 512 or 1024 on); at T = 50001, E = 256, K = 8: 29.2 us
// (1.8 TB/s; 145 us recomputing the keys in four radix passes).  Rows shorter
// than one piece, and longer ones, take an MSB-first radix select with the keys
// recomputed from global memory in each of four passes of 8-bit digits.
//
// With a counts pointer, workgroup 0 also writes MaxVio/MinVio of the step's
// counts (Eq. vio), as the stand-alone statistics kernel does: exact integer
// sum, maximum and minimum, one fp64 division each (NaN for an empty batch),
// after its own expert's selection (loading the counts at launch instead keeps
// them in registers through the selection: more spills, slower).
#include "common.h"
#include "internal.h"

#pragma clang fp contract(off)

namespace idb {

namespace {

constexpr int kQbThreads = 512;  // the global-memory kernel's workgroup
constexpr int kQbList = 4096;    // listed keys of a 512-thread workgroup
constexpr int kFewKeys = 128;    // ranked by counting
// Wanted ranks up to this many from the top are bracketed by the threads'
// largest keys (rows of up to 8192 tokens); us, with them and with a sample: T =
// 8192, E = 768, K = 10 (rank 107) 12.0 / 13.2; T = 4096, E = 64, K = 4 (rank 256)
// 11.2 / 11.3; T = 4096, E = 256, K = 24 (rank 384) 15.2 / 10.4.
constexpr int kTopRank = 160;

// Order-preserving key of a float (after -0 -> +0): a < b iff key(a) < key(b).
__device__ __forceinline__ unsigned order_key(float d) {
    const unsigned u = __float_as_uint(d + 0.0f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float key_value(unsigned o) {
    return __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o);
}

// Counts of digits into a wave's histogram.  The margins crowd into a few
// digits (the high byte is mostly sign and exponent), so runs of equal digits
// are counted in a two-entry cache and added with one LDS atomic each.
struct DigitCounter {
    unsigned d0 = 256u, c0 = 0u, d1 = 256u, c1 = 0u;  // digit 256: empty entry
    __device__ __forceinline__ void add(unsigned* h, unsigned dg) {
        if (dg == d0) {
            ++c0;
        } else if (dg == d1) {
            ++c1;
        } else {
            if (c1) atomicAdd(&h[d1], c1);
            d1 = d0;
            c1 = c0;
            d0 = dg;
            c0 = 1u;
        }
    }
    __device__ __forceinline__ void flush(unsigned* h) {
        if (c0) atomicAdd(&h[d0], c0);
        if (c1) atomicAdd(&h[d1], c1);
    }
};

// After a pass's histogram is complete, run by wave 0: the digit where the
// running count reaches kleft (lane l owns digits 4l .. 4l+3), published with
// the count of the keys below it and in it.
template <int NW>
__device__ __forceinline__ void pick_digit(unsigned (&hist)[NW][256], unsigned kleft, unsigned* pick) {
    const int lane = threadIdx.x & 63;
    unsigned c[4], tot = 0u;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        unsigned n = 0u;
#pragma unroll
        for (int w = 0; w < NW; ++w) n += hist[w][4 * lane + i];
        c[i] = n;
        tot += n;
    }
    unsigned incl = tot;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned up = __shfl_up(incl, o);
        if (lane >= o) incl += up;
    }
    unsigned run = incl - tot;  // keys in lower digits
    if (run < kleft && kleft <= incl) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (run < kleft && kleft <= run + c[i]) {
                pick[0] = (unsigned)(4 * lane + i);
                pick[1] = run;
                pick[2] = c[i];
            }
            run += c[i];
        }
    }
}

__device__ __forceinline__ void write_bias(float* bias, int j, unsigned key, float rho) {
    const float Q = -key_value(key);
    if (rho == 0.0f) {
        bias[j] = Q;
    } else {
        const float keep = rho * bias[j];
        const float take = (1.0f - rho) * Q;
        bias[j] = keep + take;
    }
}

// Radix select run by one wave over n <= 64 * V keys in LDS, which each lane
// loads once: the high bits of the key of ascending rank kleft (1-based), down
// to bit LOW and with zeros below it, a lower bound of that key, returned to
// every lane.  h: the wave's 256-bin histogram.
template <int V, int LOW>
__device__ unsigned wave_select_reg(const unsigned* vals, unsigned n, unsigned kleft, unsigned* h) {
    const int lane = threadIdx.x & 63;
    unsigned v[V];
#pragma unroll
    for (int i = 0; i < V; ++i) {
        const unsigned idx = (unsigned)lane + 64u * i;
        v[i] = idx < n ? vals[idx] : 0u;
    }
    unsigned prefix = 0u, mask = 0u;
    for (int shift = 24; shift >= LOW; shift -= 8) {
#pragma unroll
        for (int i = 0; i < 4; ++i) h[4 * lane + i] = 0u;
        wave_sync();
        DigitCounter dc;
#pragma unroll
        for (int i = 0; i < V; ++i)
            if ((unsigned)lane + 64u * i < n && (v[i] & mask) == prefix) dc.add(h, (v[i] >> shift) & 255u);
        dc.flush(h);
        wave_sync();
        unsigned c[4], tot = 0u;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            c[i] = h[4 * lane + i];
            tot += c[i];
        }
        unsigned incl = tot;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned up = __shfl_up(incl, o);
            if (lane >= o) incl += up;
        }
        unsigned run = incl - tot, digit = 0u, below = 0u;
        const bool mine = run < kleft && kleft <= incl;
        if (mine) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (run < kleft && kleft <= run + c[i]) {
                    digit = (unsigned)(4 * lane + i);
                    below = run;
                }
                run += c[i];
            }
        }
        const int src = __builtin_ctzll(__ballot(mine));
        digit = __shfl(digit, src);
        below = __shfl(below, src);
        prefix |= digit << shift;
        mask |= 255u << shift;
        kleft -= below;
        wave_sync();  // the histogram is reset by the next pass
    }
    return prefix;
}

// MaxVio, MinVio of counts whose entries i = tid + NT q (q < NQ) thread tid
// holds in n[] (0 past E), over a workgroup of NT threads.
template <int NT, int NQ>
__device__ void qb_block_stats(const int (&n)[NQ], int E, double* __restrict__ out) {
    constexpr int NW = NT / 64;
    __shared__ long long w_sum[NW];
    __shared__ int w_max[NW], w_min[NW];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    long long S = 0;
    int mx = INT32_MIN, mn = INT32_MAX;
#pragma unroll
    for (int q = 0; q < NQ; ++q)
        if (tid + NT * q < E) {
            S += n[q];
            mx = max(mx, n[q]);
            mn = min(mn, n[q]);
        }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        S += __shfl_xor(S, o);
        mx = max(mx, __shfl_xor(mx, o));
        mn = min(mn, __shfl_xor(mn, o));
    }
    if (lane == 0) {
        w_sum[wave] = S;
        w_max[wave] = mx;
        w_min[wave] = mn;
    }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < NW; ++w) {
            S += w_sum[w];
            mx = max(mx, w_max[w]);
            mn = min(mn, w_min[w]);
        }
        if (S == 0) {
            out[0] = __builtin_nan("");
            out[1] = __builtin_nan("");
        } else {
            out[0] = (double)((long long)E * mx - S) / (double)S;
            out[1] = (double)(S - (long long)E * mn) / (double)S;
        }
    }
}

// The counts that thread tid of workgroup 0 holds for qb_block_stats.
template <int NT, int NQ>
__device__ __forceinline__ void qb_stats_load(const int32_t* __restrict__ counts, int E, int (&n)[NQ]) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int i = threadIdx.x + NT * q;
        n[q] = i < E ? counts[i] : 0;
    }
}

// NT threads, R keys per thread in registers (4 <= T <= R * NT): one read of
// the row.  The wanted key is the r-th largest, r = T - k + 1.
//   1. A sample of one key per thread, spread over the row, brackets it: the
//      sample's order statistics 4 standard deviations (and 1 rank) above and 6
//      (and 5 ranks, for the Poisson tail of small ones) below the expected rank,
//      from a 16-bit radix select by one wave each (rounded outwards), give
//      [lo, hi]; no upper end where its rank would be below 1.  A bracket that
//      would fill the list (it has no room for 10 deviations of the larger K / E on
//      long rows) is narrowed to three quarters of it, still 3 deviations or
//      more to each side: T = 65536, E = 64, K = 16 29 us, where the overflowing
//      list and then the radix select took 54; T = 16384, E = 64, K = 31 16.5 / 23.8.
//      Rows of up to 8192 tokens take a cheaper bracket where r <= kTopRank (the
//      r-th largest of the threads' largest keys is a lower bound, as r keys
//      reach it), and none for r > NT, where the radix select over 16 keys per
//      thread costs less: T = 4096, E = 32, K = 16 11.2 us, 13.2 with the bracket.
//   2. The keys above hi are counted, those in [lo, hi] go to an LDS list (864
//      at T = 16384, r = 213; 3030 at T = 50001, r = 1562).
//   3. The list's histogram over 1024 equal key intervals gives the interval of
//      the wanted rank, again inside that interval while it holds many keys
//      (margins of biases that have drifted together lie close), until its few
//      keys are ranked by counting or it is a single key.
// When the bracket misses (the sample does not bind the row) or the list still
// overflows, a radix select over the registers takes over: the result is exact
// in every case.
// Bound by reading the row, then by the barriers of the three steps.
template <int NT, int R>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(NT == 512 ? 6 : 4)))
void qb_update_reg_kernel(const float* __restrict__ scores_t, const float* __restrict__ alpha, int64_t T64, int E,
                          int K, float rho, float* __restrict__ bias, const int32_t* __restrict__ counts,
                          double* __restrict__ stats) {
    constexpr int NW = NT / 64;
    constexpr int NQ = (1024 + NT - 1) / NT;  // counts per thread of workgroup 0 (E <= 1024)
    constexpr int Q = R / 4;
    constexpr int BQ = Q < 4 ? Q : 4;  // pieces in flight per batch
    constexpr int BINS = 1024;
    constexpr unsigned LIST = NT == 1024 ? 8192 : kQbList;
    static_assert(NW * 256 >= BINS, "the interval histogram shares the radix histograms' memory");
    __shared__ unsigned hist[NW][256];
    __shared__ unsigned list[LIST];
    __shared__ unsigned sample[NT];  // then the wanted interval's keys
    __shared__ unsigned pick[3];
    __shared__ unsigned nlist, nabove, nsmall, lo_s, hi_s, max_s, result_s;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int j = blockIdx.x;
    const int T = (int)T64;
    const float* row = scores_t + (int64_t)j * T;
    const bool with_stats = counts && j == 0;  // uniform over the workgroup

    // Piece p = tid + NT i holds tokens 4p .. 4p + 3; the row's last piece ends
    // at its last token and drops the tokens of the piece before it.  Slots
    // without a token hold key 0, below every key of a number.
    unsigned key[R];
    const int pieces = (T + 3) / 4;
#pragma unroll
    for (int b = 0; b < Q; b += BQ) {
        f4u sv[BQ], av[BQ];
#pragma unroll
        for (int i = 0; i < BQ; ++i) {
            const int p = tid + (b + i) * NT;
            int t0 = 4 * (p < pieces ? p : pieces - 1);
            t0 = t0 < T - 4 ? t0 : T - 4;
            sv[i] = *reinterpret_cast<const f4u*>(row + t0);
            av[i] = *reinterpret_cast<const f4u*>(alpha + t0);
        }
#pragma unroll
        for (int i = 0; i < BQ; ++i) {
#pragma unroll
            for (int c = 0; c < 4; ++c) key[4 * (b + i) + c] = order_key(sv[i].v[c] - av[i].v[c]);
            const int p = tid + (b + i) * NT;
            if (4 * p + 4 > T) {
                const int skip = p < pieces ? 4 * p + 4 - T : 4;  // leading slots without a token of their own
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (c < skip) key[4 * (b + i) + c] = 0u;
            }
        }
    }

    const unsigned k = (unsigned)((T64 * (int64_t)(E - K) + E - 1) / E);  // 1-based ascending rank
    const unsigned r_top = (unsigned)T - k + 1u;                         // the same key's rank from the top
    if (tid == 0) {
        nlist = 0u;
        nabove = 0u;
        nsmall = 0u;
        lo_s = 1u;
        hi_s = ~0u;
        max_s = 0u;
    }
    const bool whole = (unsigned)T <= LIST / 2;  // the whole row goes to the list
    const bool direct = R <= 16 && !whole && r_top > (unsigned)NT;
    if (!whole && !direct) {
        // 1. the bracket; only slots that hold a token of every thread sampled
        // (T > LIST / 2: at least one whole round of pieces)
        const bool tops = R <= 16 && r_top <= (unsigned)kTopRank;
        const int slot = tid % (4 * (T / (4 * NT)));
        unsigned mine = 0u;
        if (tops) {
#pragma unroll
            for (int r = 0; r < R; ++r) mine = key[r] > mine ? key[r] : mine;
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) mine = r == slot ? key[r] : mine;
        }
        sample[tid] = mine;
        __syncthreads();
        int hi_rank, lo_rank;  // from the top
        if (tops) {
            hi_rank = 0;
            lo_rank = (int)r_top;
        } else {
            const float share = (float)r_top / (float)T;
            const float mid = share * (float)NT, dev = sqrtf(mid * (1.0f - share));
            hi_rank = (int)(mid - 4.0f * dev - 1.0f);
            lo_rank = (int)(mid + 6.0f * dev) + 5;
            const float most = 0.75f * (float)LIST * (float)NT / (float)T;  // sampled keys
            if ((float)(lo_rank - (hi_rank > 0 ? hi_rank : 0)) > most) {
                hi_rank = (int)(mid - 0.5f * most);
                lo_rank = (int)(mid + 0.5f * most) + 1;
            }
        }
        if (wave == 0 && lo_rank <= NT) {
            const unsigned v = wave_select_reg<NT / 64, 16>(sample, (unsigned)NT, (unsigned)(NT - lo_rank + 1),
                                                            hist[0]);
            if (lane == 0 && v > 1u) lo_s = v;
        }
        if (wave == 1 && hi_rank >= 1) {
            const unsigned v = wave_select_reg<NT / 64, 16>(sample, (unsigned)NT, (unsigned)(NT - hi_rank + 1),
                                                            hist[1]);
            if (lane == 0) hi_s = v | 0xffffu;
        }
    }
    bool found = false;
    if (!direct) {
        __syncthreads();
        const unsigned lo = lo_s, hi = hi_s;
        // 2. counts above and inside, packed for one scan over the wave; one LDS
        // atomic per wave for its place in the list
        unsigned c = 0u, mx = 0u;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            c += key[r] > hi ? 0x10000u : key[r] >= lo ? 1u : 0u;
            mx = key[r] > mx ? key[r] : mx;
        }
        if (hi == ~0u) {
            // the row's largest key, one LDS atomic per wave
            auto up = [](unsigned a, unsigned b) { return a > b ? a : b; };
            mx = up(mx, (unsigned)row_rot<8>((int)mx));
            mx = up(mx, (unsigned)row_rot<4>((int)mx));
            mx = up(mx, (unsigned)row_rot<2>((int)mx));
            mx = up(mx, (unsigned)row_rot<1>((int)mx));
            const unsigned wmax = up(up((unsigned)__builtin_amdgcn_readlane((int)mx, 0),
                                        (unsigned)__builtin_amdgcn_readlane((int)mx, 16)),
                                     up((unsigned)__builtin_amdgcn_readlane((int)mx, 32),
                                        (unsigned)__builtin_amdgcn_readlane((int)mx, 48)));
            if (lane == 0) atomicMax(&max_s, wmax);
        }
        unsigned incl = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned up = __shfl_up(incl, o);
            if (lane >= o) incl += up;
        }
        unsigned base = 0u;
        if (lane == 63) {
            base = atomicAdd(&nlist, incl & 0xffffu);
            atomicAdd(&nabove, incl >> 16);
        }
        unsigned pos = __shfl(base, 63) + (incl & 0xffffu) - (c & 0xffffu);
        if ((c & 0xffffu) != 0u) {
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (key[r] >= lo && key[r] <= hi) {
                    if (pos < LIST) list[pos] = key[r];
                    ++pos;
                }
        }
        unsigned* bins = &hist[0][0];
        for (int i = tid; i < BINS; i += NT) bins[i] = 0u;
        __syncthreads();
        const unsigned n = nlist, above = nabove;
        found = above < r_top && r_top <= above + n && n <= LIST;
        if (found) {
            // 3. intervals of 2^sh keys from `from`
            unsigned want = r_top - above;  // rank from the top of the list
            unsigned from = lo, m;
            const unsigned span = (hi == ~0u ? max_s : hi) - lo;
            int sh = span < (unsigned)BINS ? 0 : 22 - __builtin_clz(span);
            unsigned width = ~0u;  // keys from `from` on that are looked at, less one
            for (;;) {
                for (unsigned i = tid; i < n; i += NT) {
                    const unsigned u = list[i];
                    if (u >= from && u - from <= width) atomicAdd(&bins[(u - from) >> sh], 1u);
                }
                __syncthreads();
                if (wave == 0) {
                    // lane l owns the 16 bins below BINS - 16 l
                    const unsigned* own = bins + BINS - 16 * (lane + 1);
                    unsigned cnt[16], tot = 0u;
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        cnt[i] = own[i];
                        tot += cnt[i];
                    }
                    unsigned sum = tot;
#pragma unroll
                    for (int o = 1; o < 64; o <<= 1) {
                        const unsigned up = __shfl_up(sum, o);
                        if (lane >= o) sum += up;
                    }
                    unsigned run = sum - tot;
                    if (run < want && want <= sum) {
#pragma unroll
                        for (int i = 15; i >= 0; --i) {
                            if (run < want && want <= run + cnt[i]) {
                                pick[0] = (unsigned)(BINS - 16 * (lane + 1) + i);
                                pick[1] = run;
                                pick[2] = cnt[i];
                            }
                            run += cnt[i];
                        }
                    }
                }
                __syncthreads();
                from += pick[0] << sh;
                want -= pick[1];
                m = pick[2];
                if (sh == 0 || m <= (unsigned)kFewKeys) break;
                // the next histogram covers this interval alone
                for (int i = tid; i < BINS; i += NT) bins[i] = 0u;
                width = (1u << sh) - 1u;
                sh = sh > 10 ? sh - 10 : 0;
                __syncthreads();
            }
            if (sh == 0) {
                if (tid == 0) result_s = from;  // one key value per interval
            } else {
                for (unsigned i = tid; i < n; i += NT) {
                    const unsigned u = list[i];
                    if (u >= from && (u - from) >> sh == 0u) sample[atomicAdd(&nsmall, 1u)] = u;
                }
                __syncthreads();
                // every thread ranks one key: the wanted one has fewer than
                // `want` keys above it and at least `want` not below it
                if (tid < (int)m) {
                    const unsigned u = sample[tid];
                    unsigned gt = 0u, ge = 0u;
                    for (unsigned i = 0; i < m; ++i) {
                        const unsigned o = sample[i];
                        gt += o > u ? 1u : 0u;
                        ge += o >= u ? 1u : 0u;
                    }
                    if (gt < want && want <= ge) result_s = u;  // equal keys write the same value
                }
            }
            __syncthreads();
            if (tid == 0) write_bias(bias, j, result_s, rho);
        }
    }
    if (!found) {
        // full radix select over the registers; the empty slots rank lowest
        unsigned kleft = k + (unsigned)(R * NT - T), prefix = 0u, mask = 0u;
        for (int shift = 24; shift >= 0; shift -= 8) {
            __syncthreads();
            for (int i = tid; i < NW * 256; i += NT) (&hist[0][0])[i] = 0u;
            __syncthreads();
            DigitCounter dc;
#pragma unroll
            for (int r = 0; r < R; ++r)
                if ((key[r] & mask) == prefix) dc.add(hist[wave], (key[r] >> shift) & 255u);
            dc.flush(hist[wave]);
            __syncthreads();
            if (wave == 0) pick_digit(hist, kleft, pick);
            __syncthreads();
            prefix |= pick[0] << shift;
            mask |= 255u << shift;
            kleft -= pick[1];
        }
        if (tid == 0) write_bias(bias, j, prefix, rho);
    }
    if (with_stats) {
        int cnt[NQ];
        qb_stats_load<NT>(counts, E, cnt);
        qb_block_stats<NT>(cnt, E, stats);
    }
}

// Any T: the keys are recomputed from global memory in every pass.
__global__ __launch_bounds__(kQbThreads) void qb_update_global_kernel(const float* __restrict__ scores_t,
                                                                      const float* __restrict__ alpha, int64_t T,
                                                                      int E, int K, float rho,
                                                                      float* __restrict__ bias,
                                                                      const int32_t* __restrict__ counts,
                                                                      double* __restrict__ stats) {
    constexpr int NW = kQbThreads / 64;
    constexpr int NQ = (1024 + kQbThreads - 1) / kQbThreads;
    __shared__ unsigned hist[NW][256];
    __shared__ unsigned pick[3];
    const int tid = threadIdx.x;
    const int wave = tid >> 6;
    const int j = blockIdx.x;
    const bool with_stats = counts && j == 0;
    int cnt[NQ];
    if (with_stats) qb_stats_load<kQbThreads>(counts, E, cnt);
    const float* row = scores_t + (int64_t)j * T;
    unsigned kleft = (unsigned)((T * (int64_t)(E - K) + E - 1) / E);
    unsigned prefix = 0u, mask = 0u;
    for (int shift = 24; shift >= 0; shift -= 8) {
        for (int i = tid; i < NW * 256; i += kQbThreads) (&hist[0][0])[i] = 0u;
        __syncthreads();
        DigitCounter dc;
        for (int64_t t = tid; t < T; t += kQbThreads) {
            const unsigned u = order_key(row[t] - alpha[t]);
            if ((u & mask) == prefix) dc.add(hist[wave], (u >> shift) & 255u);
        }
        dc.flush(hist[wave]);
        __syncthreads();
        if (wave == 0) pick_digit(hist, kleft, pick);
        __syncthreads();
        prefix |= pick[0] << shift;
        mask |= 255u << shift;
        kleft -= pick[1];
        __syncthreads();  // pick[] is rewritten by the next pass
    }
    if (tid == 0) write_bias(bias, j, prefix, rho);
    if (with_stats) qb_block_stats<kQbThreads>(cnt, E, stats);
}

template <int NT, int R>
void launch_reg(const float* scores_t, const float* alpha, int64_t T, int E, int K, float rho, float* bias,
                const int32_t* counts, double* stats, hipStream_t stream) {
    hipLaunchKernelGGL((qb_update_reg_kernel<NT, R>), dim3((unsigned)E), dim3(NT), 0, stream, scores_t, alpha, T, E, K,
                       rho, bias, counts, stats);
}

}  // namespace

hipError_t launch_qb_update(const float* scores_t, const float* alpha, int64_t T, int E, int K, float rho,
                            float* bias, const int32_t* counts, double* stats, hipStream_t stream) {
    // 512 threads while the row fits 32 keys per thread (three workgroups per
    // CU), then 1024 with up to 64; longer rows, and rows shorter than one
    // piece, are read again in every radix pass
    if (T < 4 || T > 64 * 1024)
        hipLaunchKernelGGL(qb_update_global_kernel, dim3((unsigned)E), dim3(kQbThreads), 0, stream, scores_t, alpha,
                           T, E, K, rho, bias, counts, stats);
    else if (T <= 16 * 512)
        launch_reg<512, 16>(scores_t, alpha, T, E, K, rho, bias, counts, stats, stream);
    else if (T <= 32 * 512)
        launch_reg<512, 32>(scores_t, alpha, T, E, K, rho, bias, counts, stats, stream);
    else if (T <= 32 * 1024)
        launch_reg<1024, 32>(scores_t, alpha, T, E, K, rho, bias, counts, stats, stream);
    else
        launch_reg<1024, 64>(scores_t, alpha, T, E, K, rho, bias, counts, stats, stream);
    return hipGetLastError();
}

}  // namespace idb
