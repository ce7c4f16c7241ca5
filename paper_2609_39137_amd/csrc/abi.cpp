// C ABI of the ID Balancing router step (declared in include/idb.h): argument
// checks, tiling choice and kernel launches.  Every check runs before any HIP
// call, so an invalid call enqueues nothing and touches no output.
#include "idb.h"

#include <math.h>
#include <stdarg.h>
#include <stdio.h>

#include "internal.h"

namespace {

thread_local char g_last_error[256] = "";

idb_status fail(idb_status s, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_last_error, sizeof g_last_error, fmt, ap);
    va_end(ap);
    return s;
}

idb_status hip_result(hipError_t e, const char* what) {
    if (e == hipSuccess) return IDB_OK;
    return fail(IDB_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

bool aligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

constexpr int64_t kMaxTokens = int64_t(1) << 26;
constexpr int kMaxExperts = 1024;
constexpr int kMaxSlices = 8;
constexpr int kMaxKGpu = 32;

size_t round_up(size_t n) { return (n + 255) & ~size_t(255); }

// Resolve a router variant for a shape (T tokens of E experts); returns IDB_OK and the tiling, or an error.
// one_slice: only tilings whose workgroups cover all E experts and that have
// the softmax mode (the auxiliary-loss statistics need each token's whole
// softmax in one workgroup).
idb_status resolve_tiling(int64_t T, int32_t E, idb_dtype dtype, int32_t variant, idb::RouterTiling* out,
                          bool one_slice = false) {
    const int n = idb::router_tiling_count();
    const int want_f32 = dtype == IDB_DTYPE_F32;
    const int max_slices = one_slice ? 1 : kMaxSlices;
    if (variant != 0) {
        if (variant < 1 || variant > n) return fail(IDB_ERR_INVALID_ARG, "router variant %d out of range", variant);
        idb::RouterTiling t = idb::router_tiling(variant - 1);
        if (t.is_f32 != want_f32) return fail(IDB_ERR_UNSUPPORTED, "router variant %d is for another dtype", variant);
        if (idb::router_slices(t, E) > max_slices)
            return fail(IDB_ERR_UNSUPPORTED, "router variant %d needs more than %d expert slice(s) for E=%d",
                        variant, max_slices, E);
        if (one_slice && !t.softmax)
            return fail(IDB_ERR_UNSUPPORTED, "router variant %d has no softmax mode", variant);
        *out = t;
        return IDB_OK;
    }
    // Automatic: among the tilings of this dtype, the fewest padded experts,
    // then the preferred one (the ranking follows measured throughput).
    bool found = false;
    idb::RouterTiling best{};
    long best_waste = 0;
    for (int i = 0; i < n; ++i) {
        idb::RouterTiling t = idb::router_tiling(i);
        if (t.is_f32 != want_f32) continue;
        const int ns = idb::router_slices(t, E);
        if (ns > max_slices || (one_slice && !t.softmax)) continue;
        const long waste = (long)ns * t.waves * t.we - E;
        if (!found || waste < best_waste || (waste == best_waste && t.rank < best.rank)) {
            best = t;
            best_waste = waste;
            found = true;
        }
    }
    if (!found)
        return fail(IDB_ERR_UNSUPPORTED, one_slice ? "no one-slice router tiling for E=%d" : "no router tiling for E=%d",
                    E);
    *out = idb::router_tiling_for(best, T, E);
    return IDB_OK;
}

idb_status check_router_shape(int64_t T, int32_t d, int32_t E, int32_t K, idb_dtype dtype) {
    if (dtype != IDB_DTYPE_BF16 && dtype != IDB_DTYPE_F32) return fail(IDB_ERR_INVALID_ARG, "unknown dtype %d", dtype);
    if (T < 1 || T > kMaxTokens) return fail(IDB_ERR_INVALID_ARG, "T=%lld out of [1, 2^26]", (long long)T);
    // d <= 65536 and E <= 1024 keep every operand byte offset of the fused
    // kernel (at most E * d * 4 = 2^28) inside its 32-bit buffer addressing.
    if (d < 1 || d > 65536) return fail(IDB_ERR_INVALID_ARG, "d=%d out of [1, 65536]", d);
    if (E < 1 || K < 1 || K > E) return fail(IDB_ERR_INVALID_ARG, "need 1 <= K <= E (K=%d, E=%d)", K, E);
    if (E > kMaxExperts) return fail(IDB_ERR_UNSUPPORTED, "E=%d above %d", E, kMaxExperts);
    if (E % 32 != 0) return fail(IDB_ERR_UNSUPPORTED, "E=%d is not a multiple of 32", E);
    if (K > kMaxKGpu) return fail(IDB_ERR_UNSUPPORTED, "K=%d above %d", K, kMaxKGpu);
    const int dmul = dtype == IDB_DTYPE_BF16 ? 64 : 32;
    if (d % dmul != 0) return fail(IDB_ERR_UNSUPPORTED, "d=%d is not a multiple of %d", d, dmul);
    return IDB_OK;
}

size_t router_ws_bytes(int64_t T, int32_t E, int32_t K, const idb::RouterTiling& t) {
    const int ns = idb::router_slices(t, E);
    if (ns <= 1) return 0;
    // candidates (value, score, index) [T][ns][K], then the merge's ticket
    return 3 * round_up((size_t)T * ns * K * 4) + 256;
}

// Scored path: whether the automatic choice routes this shape through
// materialised scores (scores.hip, then the selection of select.hip) instead
// of the fused tiling t.  It has small tiles for small batches and a selection
// that keeps its speed for large K, but writes and reads T x E scores, so the
// fused kernel takes over as the batch grows, and sooner the less contraction
// there is to gain from (small d).  The lines lie about where whole steps cross
// (scored / fused, us).  For K = 13 and 14 that is no sharp line: one token whose
// list overflows costs its fused tile about 10 us, so the fused time jumps with
// the data (E = 768, K = 13, d = 64: T = 8192 33 / 34, T = 16384 42 / 32, T = 24000 50 / 58).
//  - fp32: E = 256 T = 8192 45.5 / 53.9, T = 12288 60.5 / 54.5 (d = 2048); E = 128
//    T = 16384 d = 256 33.7 / 36.8, d = 64 27.0 / 24.9; E = 64 T = 32768 d = 64 29.4 / 26.7
//  - 128-expert tiles: E = 128 T = 16384 d = 2048 32.4 / 38.9, d = 64 21.9 / 21.2;
//    T = 18000, where the selection starts a second round, d = 2048 40.4 / 39.0, d = 512
//    27.1 / 25.6; E = 64 T = 20480 is level; several slices: E = 896 T = 4097 d = 64
//    K = 1 23.9 / 22.4, K = 4 26.0 / 34.5, T = 6000 K = 4 29.4 / 46.6
//  - K = 8 on 32-token tiles: d = 2048 E = 768 T = 2048 27.2 / 34.1, T = 2560 31.2 /
//    33.9, T = 4096 37.2 / 35.0; E = 256 T = 2560 22.6 / 25.5, T = 4096 28.1 / 26.5;
//    d = 512 E = 768 T = 1024 17.3 / 18.9, T = 2048 21.4 / 19.3
//  - K > 12 (the fused lists overflow from about K = 14 on, the slice merge
//    grows): 384-expert tiles: K = 16 E = 768 T = 16384 d = 2048 71 / 139, E = 384
//    T = 65536 d = 64 65 / 171; K = 14 E = 384 T = 24000 d = 64 42 / 49, d = 4096 129 / 103;
//    K = 13 E = 384 T = 8192 d = 1024 32 / 26, T = 32768 56 / 51; K = 13 E = 768 T =
//    32768 d = 2048 124 / 134, T = 65536 d = 1024 181 / 163, d = 64 85 / 98.  256-expert
//    tiles: K = 16 one slice, E = 256 T = 12000 d = 64 28.9 / 27.7; four slices, E = 1024
//    T = 12000 K = 13 d = 256 53.9 / 68.4.  K > 20: E = 256 T = 16384 K = 21 d = 1024 39 / 138,
//    E = 1024 T = 16384 K = 32 d = 256 73 / 954
//  - a row-major router matrix, which the fused kernels read at a quarter to
//    half of the packed rate and the scored path packs first: K = 8, d = 1024
//    E = 256 T = 16384 35 / 35, E = 768 T = 8192 39 / 43, E = 1024 T = 6000 40 / 48;
//    d = 768 E = 256 T = 12000 31 / 29, E = 768 T = 8192 37 / 37; d = 384 E = 256 T = 8192
//    24 / 22, E = 768 T = 2561 25 / 26, T = 8192 37 / 29; d = 256 E = 768 T = 3000 25.0 / 23.5
bool use_scores(int64_t T, int32_t d, int32_t E, int32_t K, const idb::RouterTiling& t, bool row_major) {
    constexpr int64_t kMi = int64_t(1) << 20;
    const int64_t n = T * E;
    if (n > 64 * kMi) return false;  // 256 MB of scores
    const bool one_slice = idb::router_slices(t, E) <= 1;
    if (t.is_f32) return n <= (d >= 256 ? 2 * kMi : 3 * kMi / 2);
    if (t.id == 4) {
        if (E <= 64) return T <= 20480;
        if (E <= 128) return T <= (d >= 256 ? 16384 : 14336);
        return n <= (K > 1 ? 6 * kMi : 3 * kMi);
    }
    if (K > 12) {
        if (K > 20) return true;
        if (!idb::tiling_is_16(t)) return n <= (one_slice ? 3 * kMi : 12 * kMi);
        if (one_slice) return K > (d >= 2048 ? 14 : 13) || n <= 3 * kMi;
        return K > 13 || d < 1024 || n <= 32 * kMi;
    }
    if (row_major && d >= 384 && n <= (d >= 768 ? 6 * kMi : 2 * kMi)) return true;
    return T <= (d >= 1024 ? 2560 : 1280);
}

// From this many tokens on the scored path packs a row-major router matrix
// into its workspace first.  Whole steps, packed first / row-major, us, K = 8: the
// larger the matrix and the more token tiles read it, the more the pack gives (E
// = 1024, d = 4096: T = 777 39.5 / 54.5, T = 2560 57.4 / 86.1; E = 256, d = 4096: T = 777
// 24.2 / 21.1, T = 1280 25.7 / 31.4; E = 768, d = 1024: T = 1024 23.7 / 21.1, T = 2560 29.0 /
// 32.6), and a small matrix pays for the launch alone (E = 256, d = 256: T = 1024
// 14.7 / 13.0, T = 2560 17.8 / 17.8; E = 64, d = 256: T = 2560 13.5 / 11.7): one line for
// all of them.  Not fp32, whose MFMAs take long enough to cover the loads (T =
// 4096, d = 256, E = 64: score kernel 7.4 us unpacked, 8.4 packed).
constexpr int64_t kPackTokens = 1024;

bool packs_first(int64_t T, idb_dtype dtype) { return T >= kPackTokens && dtype == IDB_DTYPE_BF16; }

size_t weight_bytes(int32_t E, int32_t d) { return (size_t)E * d * 2; }

// Its workspace: the scores [T][E], the ticket, then (when there is room) the
// packed router matrix.
size_t score_ws_bytes(int64_t T, int32_t E) { return round_up((size_t)T * E * 4) + 256; }

// Auxiliary-loss statistics: per-tile softmax column sums [tiles][E] fp32,
// per-tile counts [tiles][E] int32, kAuxMaxBlocks block records, the ticket.
size_t aux_rows_bytes(int64_t T, int32_t E, const idb::RouterTiling& t) {
    return round_up((size_t)((T + t.bt - 1) / t.bt) * E * 4);
}
size_t aux_ws_bytes(int64_t T, int32_t E, const idb::RouterTiling& t) {
    return 2 * aux_rows_bytes(T, E, t) + round_up(idb::kAuxMaxBlocks * sizeof(idb::AuxPartial)) + 256;
}

struct RouterCall {
    idb::RouterTiling tiling;
    idb::RouterArgs args;
    unsigned* ticket;  // the merge's (multi-slice tilings) or the statistics kernel's ticket
    idb::AuxPartial* aux_partial;  // auxiliary-loss statistics: block records
    bool scored;                   // the scored path: launch_scores, then launch_select_step
    float* scores;                 // scored: the [T][E] scores in the workspace
    char* pack_to;                 // scored: nullable, where a row-major router matrix is packed first
};

idb_status prepare_router(const void* x, const void* W_g, idb_dtype dtype, idb_weight_layout layout,
                          const float* bias, int64_t T, int32_t d,
                          int32_t E, int32_t K, int32_t* expert_idx, float* gate_w, int32_t* counts,
                          int32_t accumulate_counts, float* scores_dump, void* workspace, size_t workspace_bytes,
                          int32_t variant, bool need_inputs, RouterCall* call, bool qb = false,
                          bool aux = false, bool whole = false) {
    // whole: the call makes all of the step's launches itself, so it accepts
    // IDB_ROUTER_AUTO_SCORES (the split calls refuse it: their second launch
    // could not tell which path the first one took).  Only that choice uses
    // more of the workspace than the tiling's own part: a caller of variant 0
    // may keep other data there, or share it between streams where the tiling
    // needs none.
    const bool own_workspace = whole && variant == IDB_ROUTER_AUTO_SCORES;
    if (own_workspace) variant = IDB_ROUTER_AUTO;
    // Quantile Balancing keeps K + 1 candidates per token (the (K+1)-th is the cutoff)
    const int32_t KL = qb ? K + 1 : K;
    idb_status st = check_router_shape(T, d, E, KL, dtype);
    if (st != IDB_OK) return st;
    if (layout != IDB_WEIGHT_ROW_MAJOR && layout != IDB_WEIGHT_PACKED)
        return fail(IDB_ERR_INVALID_ARG, "unknown weight layout %d", layout);
    if (need_inputs) {
        if (!x || !W_g || (!bias && !aux)) return fail(IDB_ERR_INVALID_ARG, "null input pointer");
        if (!aligned(x, 16) || !aligned(W_g, 16)) return fail(IDB_ERR_INVALID_ARG, "x and W_g must be 16-byte aligned");
        if (bias && !aligned(bias, 4)) return fail(IDB_ERR_INVALID_ARG, "bias must be 4-byte aligned");
        if (scores_dump && !aligned(scores_dump, 16))
            return fail(IDB_ERR_INVALID_ARG, "scores_dump must be 16-byte aligned");
    }
    if (!expert_idx || !gate_w || !counts) return fail(IDB_ERR_INVALID_ARG, "null output pointer");
    if (!aligned(expert_idx, 4) || !aligned(gate_w, 4) || !aligned(counts, 4))
        return fail(IDB_ERR_INVALID_ARG, "outputs must be 4-byte aligned");
    st = resolve_tiling(T, E, dtype, variant, &call->tiling, aux);
    if (st != IDB_OK) return st;
    const size_t need = aux ? aux_ws_bytes(T, E, call->tiling) : router_ws_bytes(T, E, KL, call->tiling);
    if (need > 0) {
        if (!workspace || workspace_bytes < need)
            return fail(IDB_ERR_INVALID_ARG, "workspace of %zu bytes needed, %zu given", need, workspace_bytes);
        if (!aligned(workspace, 16)) return fail(IDB_ERR_INVALID_ARG, "workspace must be 16-byte aligned");
    }
    idb::RouterArgs& a = call->args;
    a.x = x;
    a.W = W_g;
    a.w_packed = layout == IDB_WEIGHT_PACKED;
    a.bias = bias;
    a.T = T;
    a.d = d;
    a.E = E;
    a.K = K;
    a.idx = expert_idx;
    a.w = gate_w;
    a.counts = counts;
    a.dump = scores_dump;
    const int ns = idb::router_slices(call->tiling, E);
    a.zero_counts = (!accumulate_counts && ns > 1) ? 1 : 0;
    const size_t part = round_up((size_t)T * ns * KL * 4);
    char* ws = static_cast<char*>(workspace);
    a.cand_v = need ? reinterpret_cast<float*>(ws) : nullptr;
    a.cand_s = need ? reinterpret_cast<float*>(ws + part) : nullptr;
    a.cand_i = need ? reinterpret_cast<int32_t*>(ws + 2 * part) : nullptr;
    // the merge's ticket slot; the router kernel's first workgroup zeroes it,
    // so a merge that applies the controller update may follow any router call
    a.ticket = need ? reinterpret_cast<unsigned*>(ws + 3 * part) : nullptr;
    a.alpha = nullptr;
    a.scores_t = nullptr;
    a.softmax = aux ? 1 : 0;
    a.prob_part = nullptr;
    a.cnt_part = nullptr;
    call->ticket = need ? reinterpret_cast<unsigned*>(ws + 3 * part) : nullptr;
    call->aux_partial = nullptr;
    // The scored path may need more scratch than the fused tiling: a workspace
    // that was sized for another batch keeps the fused one.
    const size_t scored_need = score_ws_bytes(T, E);
    call->scored = own_workspace && workspace && aligned(workspace, 16) && workspace_bytes >= scored_need &&
                   use_scores(T, d, E, K, call->tiling, layout == IDB_WEIGHT_ROW_MAJOR);
    call->pack_to = nullptr;
    call->scores = nullptr;
    if (call->scored) {
        call->scores = reinterpret_cast<float*>(ws);
        call->ticket = reinterpret_cast<unsigned*>(ws + scored_need - 256);
        a.ticket = call->ticket;
        a.zero_counts = accumulate_counts ? 0 : 1;
        a.cand_v = a.cand_s = nullptr;
        a.cand_i = nullptr;
        if (layout == IDB_WEIGHT_ROW_MAJOR && packs_first(T, dtype) &&
            workspace_bytes - scored_need >= weight_bytes(E, d))
            call->pack_to = ws + scored_need;
    }
    if (aux) {
        // one slice: no candidates; the statistics' per-tile rows instead
        const size_t rows = aux_rows_bytes(T, E, call->tiling);
        a.bias = nullptr;
        a.cand_v = a.cand_s = nullptr;
        a.cand_i = nullptr;
        a.prob_part = reinterpret_cast<float*>(ws);
        a.cnt_part = reinterpret_cast<int32_t*>(ws + rows);
        call->aux_partial = reinterpret_cast<idb::AuxPartial*>(ws + 2 * rows);
        call->ticket =
            reinterpret_cast<unsigned*>(ws + 2 * rows + round_up(idb::kAuxMaxBlocks * sizeof(idb::AuxPartial)));
        a.ticket = call->ticket;  // zeroed by the router kernel, taken by the statistics kernel
    }
    return IDB_OK;
}

idb_status enqueue_score_select(const RouterCall& c, int32_t accumulate_counts, hipStream_t stream,
                                hipEvent_t start = nullptr, hipEvent_t stop = nullptr) {
    if (c.scored) {
        idb::RouterArgs a = c.args;
        if (c.pack_to) {
            idb_status st = hip_result(idb::launch_pack_weight(a.W, c.pack_to, a.E, (int64_t)a.d * 2, stream),
                                       "pack weight launch");
            if (st != IDB_OK) return st;
            a.W = c.pack_to;
            a.w_packed = 1;
        }
        return hip_result(idb::launch_scores(c.tiling, a, c.scores, stream), "router score launch");
    }
    const int ns = idb::router_slices(c.tiling, c.args.E);
    if (ns <= 1 && !accumulate_counts && !c.args.cnt_part) {
        idb_status st = hip_result(idb::launch_fill_i32(c.args.counts, 0, c.args.E, stream), "zero counts");
        if (st != IDB_OK) return st;
    }
    return hip_result(idb::launch_router_score_select(c.tiling, c.args, stream, start, stop),
                      "router score/select launch");
}

}  // namespace

extern "C" {

size_t idb_router_workspace_bytes(int64_t T, int32_t d, int32_t E, int32_t K, idb_dtype dtype, int32_t variant) {
    if (check_router_shape(T, d, E, K, dtype) != IDB_OK) return 0;
    const bool own_workspace = variant == IDB_ROUTER_AUTO_SCORES;
    idb::RouterTiling t;
    if (resolve_tiling(T, E, dtype, own_workspace ? IDB_ROUTER_AUTO : variant, &t) != IDB_OK) return 0;
    const size_t fused = router_ws_bytes(T, E, K, t);
    // room for the path either weight layout may take
    if (!own_workspace || !(use_scores(T, d, E, K, t, false) || use_scores(T, d, E, K, t, true))) return fused;
    const size_t scored = score_ws_bytes(T, E) + (packs_first(T, dtype) ? weight_bytes(E, d) : 0);
    return scored > fused ? scored : fused;
}

int32_t idb_router_uses_scores(int64_t T, int32_t d, int32_t E, int32_t K, idb_dtype dtype,
                               idb_weight_layout weight_layout, size_t workspace_bytes, int32_t variant) {
    idb::RouterTiling t;
    if (variant != IDB_ROUTER_AUTO_SCORES || check_router_shape(T, d, E, K, dtype) != IDB_OK ||
        resolve_tiling(T, E, dtype, IDB_ROUTER_AUTO, &t) != IDB_OK)
        return 0;
    return workspace_bytes >= score_ws_bytes(T, E) && use_scores(T, d, E, K, t, weight_layout == IDB_WEIGHT_ROW_MAJOR);
}

idb_status idb_router_variant_info(int64_t T, int32_t d, int32_t E, int32_t K, idb_dtype dtype, int32_t variant,
                                   int32_t out[5]) {
    if (!out) return fail(IDB_ERR_INVALID_ARG, "null out");
    idb_status st = check_router_shape(T, d, E, K, dtype);
    if (st != IDB_OK) return st;
    idb::RouterTiling t;
    st = resolve_tiling(T, E, dtype, variant, &t);
    if (st != IDB_OK) return st;
    out[0] = t.bt;
    out[1] = idb::router_slices(t, E);
    out[2] = t.waves;
    out[3] = t.we;
    out[4] = t.id;
    return IDB_OK;
}

idb_status idb_router_score_select(const void* x, const void* W_g, idb_dtype dtype, idb_weight_layout weight_layout,
                                   const float* bias, int64_t T, int32_t d, int32_t E, int32_t K, int32_t* expert_idx,
                                   float* gate_w, int32_t* counts, int32_t accumulate_counts, float* scores_dump,
                                   void* workspace, size_t workspace_bytes, int32_t variant, hipStream_t stream) {
    RouterCall c;
    idb_status st = prepare_router(x, W_g, dtype, weight_layout, bias, T, d, E, K, expert_idx, gate_w, counts, accumulate_counts,
                                   scores_dump, workspace, workspace_bytes, variant, true, &c);
    if (st != IDB_OK) return st;
    return enqueue_score_select(c, accumulate_counts, stream);
}

idb_status idb_router_score_select_timed(const void* x, const void* W_g, idb_dtype dtype,
                                         idb_weight_layout weight_layout, const float* bias, int64_t T, int32_t d,
                                         int32_t E, int32_t K, int32_t* expert_idx, float* gate_w, int32_t* counts,
                                         int32_t accumulate_counts, float* scores_dump, void* workspace,
                                         size_t workspace_bytes, int32_t variant, hipStream_t stream,
                                         hipEvent_t start_event, hipEvent_t stop_event) {
    RouterCall c;
    idb_status st = prepare_router(x, W_g, dtype, weight_layout, bias, T, d, E, K, expert_idx, gate_w, counts, accumulate_counts,
                                   scores_dump, workspace, workspace_bytes, variant, true, &c);
    if (st != IDB_OK) return st;
    return enqueue_score_select(c, accumulate_counts, stream, start_event, stop_event);
}

idb_status idb_router_merge(int64_t T, int32_t d, int32_t E, int32_t K, idb_dtype dtype, int32_t* expert_idx,
                            float* gate_w, int32_t* counts, void* workspace, size_t workspace_bytes, int32_t variant,
                            hipStream_t stream) {
    RouterCall c;
    idb_status st = prepare_router(nullptr, nullptr, dtype, IDB_WEIGHT_ROW_MAJOR, nullptr, T, d, E, K, expert_idx, gate_w, counts, 1,
                                   nullptr, workspace, workspace_bytes, variant, false, &c);
    if (st != IDB_OK) return st;
    return hip_result(idb::launch_router_merge(c.tiling, c.args, nullptr, stream), "router merge launch");
}

idb_status idb_router_forward(const void* x, const void* W_g, idb_dtype dtype, idb_weight_layout weight_layout,
                              const float* bias, int64_t T, int32_t d, int32_t E, int32_t K, int32_t* expert_idx,
                              float* gate_w, int32_t* counts, int32_t accumulate_counts, float* scores_dump,
                              void* workspace, size_t workspace_bytes, int32_t variant, hipStream_t stream) {
    RouterCall c;
    idb_status st = prepare_router(x, W_g, dtype, weight_layout, bias, T, d, E, K, expert_idx, gate_w, counts, accumulate_counts,
                                   scores_dump, workspace, workspace_bytes, variant, true, &c, false, false, true);
    if (st != IDB_OK) return st;
    st = enqueue_score_select(c, accumulate_counts, stream);
    if (st != IDB_OK) return st;
    if (c.scored) return hip_result(idb::launch_select_step(c.args, c.scores, nullptr, stream), "select launch");
    return hip_result(idb::launch_router_merge(c.tiling, c.args, nullptr, stream), "router merge launch");
}

size_t idb_router_packed_weight_bytes(int32_t E, int32_t d, idb_dtype dtype) {
    if (check_router_shape(1, d, E, 1, dtype) != IDB_OK) return 0;
    return (size_t)E * d * (dtype == IDB_DTYPE_BF16 ? 2 : 4);
}

idb_status idb_router_pack_weight(const void* W_g, idb_dtype dtype, int32_t E, int32_t d, void* W_packed,
                                  hipStream_t stream) {
    idb_status st = check_router_shape(1, d, E, 1, dtype);
    if (st != IDB_OK) return st;
    if (!W_g || !W_packed) return fail(IDB_ERR_INVALID_ARG, "null pointer");
    if (!aligned(W_g, 16) || !aligned(W_packed, 16)) return fail(IDB_ERR_INVALID_ARG, "W_g and W_packed must be 16-byte aligned");
    const size_t bytes = (size_t)E * d * (dtype == IDB_DTYPE_BF16 ? 2 : 4);
    const char* a0 = static_cast<const char*>(W_g);
    const char* b0 = static_cast<const char*>(W_packed);
    if (a0 < b0 + bytes && b0 < a0 + bytes) return fail(IDB_ERR_INVALID_ARG, "W_packed overlaps W_g");
    const int64_t rb = (int64_t)d * (dtype == IDB_DTYPE_BF16 ? 2 : 4);
    return hip_result(idb::launch_pack_weight(W_g, W_packed, E, rb, stream), "pack weight launch");
}

idb_status idb_select_from_scores(const float* scores, const float* bias, int64_t T, int32_t E, int32_t K,
                                  int32_t* expert_idx, float* gate_w, int32_t* counts, int32_t accumulate_counts,
                                  hipStream_t stream) {
    if (!scores || !bias || !expert_idx || !gate_w || !counts) return fail(IDB_ERR_INVALID_ARG, "null pointer");
    if (T < 1 || T > kMaxTokens) return fail(IDB_ERR_INVALID_ARG, "T=%lld out of [1, 2^26]", (long long)T);
    if (E < 1 || K < 1 || K > E) return fail(IDB_ERR_INVALID_ARG, "need 1 <= K <= E (K=%d, E=%d)", K, E);
    if (E > kMaxExperts) return fail(IDB_ERR_UNSUPPORTED, "E=%d above %d", E, kMaxExperts);
    if (K > kMaxKGpu) return fail(IDB_ERR_UNSUPPORTED, "K=%d above %d", K, kMaxKGpu);
    if (!aligned(scores, 4) || !aligned(bias, 4) || !aligned(expert_idx, 4) || !aligned(gate_w, 4) ||
        !aligned(counts, 4))
        return fail(IDB_ERR_INVALID_ARG, "buffers must be 4-byte aligned");
    if (!accumulate_counts) {
        idb_status st = hip_result(idb::launch_fill_i32(counts, 0, E, stream), "zero counts");
        if (st != IDB_OK) return st;
    }
    return hip_result(idb::launch_select_from_scores(scores, bias, T, E, K, expert_idx, gate_w, counts, stream),
                      "select launch");
}

namespace {
idb_status check_controller(const idb_controller_cfg* cfg, const idb_controller_state* state, const double* stats) {
    if (!cfg || !state) return fail(IDB_ERR_INVALID_ARG, "null pointer");
    if (!state->bias || !state->e_prev || !state->step || !state->status)
        return fail(IDB_ERR_INVALID_ARG, "null state buffer");
    if (cfg->E < 1 || cfg->E > kMaxExperts) return fail(IDB_ERR_INVALID_ARG, "E=%d out of [1, 1024]", cfg->E);
    if (!(cfg->Ki >= 0.0f) || !(cfg->Kd >= 0.0f) || !isfinite(cfg->Ki) || !isfinite(cfg->Kd))
        return fail(IDB_ERR_INVALID_ARG, "gains must be finite and >= 0");
    if (cfg->integral_mode != IDB_INTEGRAL_ERROR && cfg->integral_mode != IDB_INTEGRAL_SIGN)
        return fail(IDB_ERR_INVALID_ARG, "unknown integral mode %d", cfg->integral_mode);
    if (cfg->center != 0 && cfg->center != 1) return fail(IDB_ERR_INVALID_ARG, "center must be 0 or 1");
    if (!aligned(state->bias, 4) || !aligned(state->e_prev, 4) || !aligned(state->step, 8) ||
        !aligned(state->status, 4) || (stats && !aligned(stats, 8)))
        return fail(IDB_ERR_INVALID_ARG, "misaligned buffer");
    return IDB_OK;
}

idb_status enqueue_controller(const int32_t* counts, const idb_controller_cfg* cfg, const idb_controller_state* state,
                              double* stats, hipStream_t stream) {
    return hip_result(idb::launch_controller_update(counts, cfg->E, cfg->Ki, cfg->Kd,
                                                    cfg->integral_mode == IDB_INTEGRAL_SIGN, cfg->center,
                                                    state->bias, state->e_prev, state->step, state->status, stats,
                                                    stream),
                      "controller launch");
}

idb_status controller_call(const int32_t* counts, const idb_controller_cfg* cfg, const idb_controller_state* state,
                           double* stats, hipStream_t stream) {
    if (!counts) return fail(IDB_ERR_INVALID_ARG, "null pointer");
    idb_status st = check_controller(cfg, state, stats);
    if (st != IDB_OK) return st;
    if (!aligned(counts, 4)) return fail(IDB_ERR_INVALID_ARG, "misaligned buffer");
    return enqueue_controller(counts, cfg, state, stats, stream);
}
// The second launch of idb_router_step: the slice merge whose last workgroup
// applies the update (multi-slice tilings), or the controller step launch
// (one-slice tilings, whose router kernel finished the counts itself).
idb_status enqueue_merge_step(const RouterCall& c, const idb_controller_cfg* cfg, const idb_controller_state* state,
                              double* out_maxvio_minvio, hipStream_t stream) {
    if (!c.ticket) return enqueue_controller(c.args.counts, cfg, state, out_maxvio_minvio, stream);
    idb::CtrlArgs k;
    k.Ki = cfg->Ki;
    k.Kd = cfg->Kd;
    k.sign_mode = cfg->integral_mode == IDB_INTEGRAL_SIGN;
    k.center = cfg->center;
    k.bias = state->bias;
    k.e_prev = state->e_prev;
    k.step = state->step;
    k.status = state->status;
    k.stats = out_maxvio_minvio;
    k.ticket = c.ticket;
    if (c.scored) return hip_result(idb::launch_select_step(c.args, c.scores, &k, stream), "select launch");
    return hip_result(idb::launch_router_merge(c.tiling, c.args, &k, stream), "router merge launch");
}


}  // namespace

idb_status idb_controller_update(const int32_t* counts, const idb_controller_cfg* cfg,
                                 const idb_controller_state* state, hipStream_t stream) {
    return controller_call(counts, cfg, state, nullptr, stream);
}

idb_status idb_controller_step(const int32_t* counts, const idb_controller_cfg* cfg,
                               const idb_controller_state* state, double* out_maxvio_minvio, hipStream_t stream) {
    if (!out_maxvio_minvio) return fail(IDB_ERR_INVALID_ARG, "null statistics output");
    return controller_call(counts, cfg, state, out_maxvio_minvio, stream);
}

idb_status idb_router_step(const void* x, const void* W_g, idb_dtype dtype, idb_weight_layout weight_layout,
                           int64_t T, int32_t d, int32_t K, const idb_controller_cfg* cfg,
                           const idb_controller_state* state, int32_t* expert_idx, float* gate_w, int32_t* counts,
                           int32_t accumulate_counts, double* out_maxvio_minvio, void* workspace,
                           size_t workspace_bytes, int32_t variant, hipStream_t stream) {
    idb_status st = check_controller(cfg, state, out_maxvio_minvio);
    if (st != IDB_OK) return st;
    RouterCall c;
    st = prepare_router(x, W_g, dtype, weight_layout, state->bias, T, d, cfg->E, K, expert_idx, gate_w, counts,
                        accumulate_counts, nullptr, workspace, workspace_bytes, variant, true, &c, false, false, true);
    if (st != IDB_OK) return st;
    st = enqueue_score_select(c, accumulate_counts, stream);
    if (st != IDB_OK) return st;
    return enqueue_merge_step(c, cfg, state, out_maxvio_minvio, stream);
}

idb_status idb_router_merge_step(int64_t T, int32_t d, int32_t K, idb_dtype dtype, const idb_controller_cfg* cfg,
                                 const idb_controller_state* state, int32_t* expert_idx, float* gate_w,
                                 int32_t* counts, double* out_maxvio_minvio, void* workspace, size_t workspace_bytes,
                                 int32_t variant, hipStream_t stream) {
    idb_status st = check_controller(cfg, state, out_maxvio_minvio);
    if (st != IDB_OK) return st;
    RouterCall c;
    st = prepare_router(nullptr, nullptr, dtype, IDB_WEIGHT_ROW_MAJOR, nullptr, T, d, cfg->E, K, expert_idx, gate_w,
                        counts, 1, nullptr, workspace, workspace_bytes, variant, false, &c);
    if (st != IDB_OK) return st;
    return enqueue_merge_step(c, cfg, state, out_maxvio_minvio, stream);
}

idb_status idb_router_step_noalloc(const void* x, const void* W_g, idb_dtype dtype, idb_weight_layout weight_layout,
                                   int64_t T, int32_t d, int32_t K, const idb_controller_cfg* cfg,
                                   const idb_controller_state* state, int32_t* expert_idx, float* gate_w,
                                   int32_t* counts, int32_t accumulate_counts, double* out_maxvio_minvio,
                                   int32_t variant, hipStream_t stream) {
    // every argument check of idb_router_step first, without any HIP call
    idb_status st = check_controller(cfg, state, out_maxvio_minvio);
    if (st != IDB_OK) return st;
    st = check_router_shape(T, d, cfg->E, K, dtype);
    if (st != IDB_OK) return st;
    idb::RouterTiling t;
    st = resolve_tiling(T, cfg->E, dtype, variant, &t);
    if (st != IDB_OK) return st;
    const size_t need = router_ws_bytes(T, cfg->E, K, t);
    const size_t have = idb::noalloc_scratch_bytes();
    if (need > have)
        return fail(IDB_ERR_UNSUPPORTED,
                    "idb_router_step_noalloc: this shape needs %zu bytes of scratch, the fixed scratch holds %zu "
                    "(T=%lld, E=%d, K=%d; use idb_router_step with a workspace)",
                    need, have, (long long)T, cfg->E, K);
    {
        // pointers, alignment and layout as idb_router_step checks them; the
        // workspace stands in as an aligned placeholder (only its size and
        // alignment are checked, nothing is dereferenced)
        RouterCall probe;
        st = prepare_router(x, W_g, dtype, weight_layout, state->bias, T, d, cfg->E, K, expert_idx, gate_w, counts,
                            accumulate_counts, nullptr, reinterpret_cast<void*>(uintptr_t(256)), have, variant, true,
                            &probe);
        if (st != IDB_OK) return st;
    }
    void* ws = nullptr;
    // one-slice tilings need no scratch and keep to the fused kernel: their
    // calls may overlap on a device, which sharing the array would forbid; the
    // others have the whole array to themselves
    if (need > 0) {
        if (variant == IDB_ROUTER_AUTO) variant = IDB_ROUTER_AUTO_SCORES;
        int dev = -1;
        st = hip_result(hipGetDevice(&dev), "current device");
        if (st != IDB_OK) return st;
        if (stream) {
            hipDevice_t sdev = -1;
            st = hip_result(hipStreamGetDevice(stream, &sdev), "stream device");
            if (st != IDB_OK) return st;
            if ((int)sdev != dev)
                return fail(IDB_ERR_INVALID_ARG, "stream belongs to device %d, current device is %d", (int)sdev, dev);
        }
        st = hip_result(idb::noalloc_scratch(dev, &ws), "scratch address");
        if (st != IDB_OK) return st;
    }
    return idb_router_step(x, W_g, dtype, weight_layout, T, d, K, cfg, state, expert_idx, gate_w, counts,
                           accumulate_counts, out_maxvio_minvio, ws, need > 0 ? have : 0, variant, stream);
}

size_t idb_qb_router_workspace_bytes(int64_t T, int32_t d, int32_t E, int32_t K, idb_dtype dtype,
                                     int32_t variant) {
    if (K < 1 || check_router_shape(T, d, E, K + 1, dtype) != IDB_OK) return 0;
    idb::RouterTiling t;
    if (resolve_tiling(T, E, dtype, variant, &t) != IDB_OK) return 0;
    return router_ws_bytes(T, E, K + 1, t);
}

idb_status idb_qb_router_forward(const void* x, const void* W_g, idb_dtype dtype, idb_weight_layout weight_layout,
                                 const float* bias, int64_t T, int32_t d, int32_t E, int32_t K, int32_t* expert_idx,
                                 float* gate_w, int32_t* counts, int32_t accumulate_counts, float* scores_t,
                                 float* alpha, void* workspace, size_t workspace_bytes, int32_t variant,
                                 hipStream_t stream) {
    if (K < 1) return fail(IDB_ERR_INVALID_ARG, "K=%d below 1", K);
    if (K + 1 > E) return fail(IDB_ERR_INVALID_ARG, "Quantile Balancing needs K + 1 <= E (K=%d, E=%d)", K, E);
    if (!scores_t || !alpha) return fail(IDB_ERR_INVALID_ARG, "null scores_t or alpha");
    if (!aligned(scores_t, 4) || !aligned(alpha, 4)) return fail(IDB_ERR_INVALID_ARG, "misaligned scores_t or alpha");
    RouterCall c;
    idb_status st = prepare_router(x, W_g, dtype, weight_layout, bias, T, d, E, K, expert_idx, gate_w, counts,
                                   accumulate_counts, nullptr, workspace, workspace_bytes, variant, true, &c, true);
    if (st != IDB_OK) return st;
    c.args.alpha = alpha;
    c.args.scores_t = scores_t;
    st = enqueue_score_select(c, accumulate_counts, stream);
    if (st != IDB_OK) return st;
    return hip_result(idb::launch_router_merge(c.tiling, c.args, nullptr, stream), "router merge launch");
}

idb_status idb_qb_update(const float* scores_t, const float* alpha, int64_t T, int32_t E, int32_t K, float rho,
                         float* bias, const int32_t* counts, double* out_maxvio_minvio, hipStream_t stream) {
    if (!scores_t || !alpha || !bias) return fail(IDB_ERR_INVALID_ARG, "null pointer");
    if (!counts != !out_maxvio_minvio)
        return fail(IDB_ERR_INVALID_ARG, "counts and out_maxvio_minvio go together (both or neither)");
    if (T < 1 || T > kMaxTokens) return fail(IDB_ERR_INVALID_ARG, "T=%lld out of [1, 2^26]", (long long)T);
    if (E < 2 || E > kMaxExperts) return fail(IDB_ERR_INVALID_ARG, "E=%d out of [2, %d]", E, kMaxExperts);
    if (K < 1 || K >= E) return fail(IDB_ERR_INVALID_ARG, "need 1 <= K < E (K=%d, E=%d)", K, E);
    if (!(rho >= 0.0f && rho < 1.0f)) return fail(IDB_ERR_INVALID_ARG, "rho must lie in [0, 1)");
    if (!aligned(scores_t, 4) || !aligned(alpha, 4) || !aligned(bias, 4) || !aligned(counts, 4) ||
        !aligned(out_maxvio_minvio, 8))
        return fail(IDB_ERR_INVALID_ARG, "misaligned buffer");
    return hip_result(idb::launch_qb_update(scores_t, alpha, T, E, K, rho, bias, counts, out_maxvio_minvio, stream),
                      "Quantile Balancing launch");
}

size_t idb_aux_router_workspace_bytes(int64_t T, int32_t d, int32_t E, int32_t K, idb_dtype dtype,
                                      int32_t variant) {
    if (check_router_shape(T, d, E, K, dtype) != IDB_OK) return 0;
    idb::RouterTiling t;
    if (resolve_tiling(T, E, dtype, variant, &t, true) != IDB_OK) return 0;
    return aux_ws_bytes(T, E, t);
}

idb_status idb_aux_router_forward(const void* x, const void* W_g, idb_dtype dtype, idb_weight_layout weight_layout,
                                  int64_t T, int32_t d, int32_t E, int32_t K, double alpha, int32_t* expert_idx,
                                  float* gate_w, int32_t* counts, double* f, double* P, double* loss,
                                  double* out_maxvio_minvio, float* logits_dump, void* workspace,
                                  size_t workspace_bytes, int32_t variant, hipStream_t stream) {
    if (!f || !P || !loss) return fail(IDB_ERR_INVALID_ARG, "null statistics output");
    if (!aligned(f, 8) || !aligned(P, 8) || !aligned(loss, 8) ||
        (out_maxvio_minvio && !aligned(out_maxvio_minvio, 8)))
        return fail(IDB_ERR_INVALID_ARG, "statistics outputs must be 8-byte aligned");
    if (!isfinite(alpha)) return fail(IDB_ERR_INVALID_ARG, "alpha must be finite");
    RouterCall c;
    idb_status st = prepare_router(x, W_g, dtype, weight_layout, nullptr, T, d, E, K, expert_idx, gate_w, counts, 0,
                                   logits_dump, workspace, workspace_bytes, variant, true, &c, false, true);
    if (st != IDB_OK) return st;
    st = enqueue_score_select(c, 0, stream);
    if (st != IDB_OK) return st;
    const int64_t tiles = (T + c.tiling.bt - 1) / c.tiling.bt;  // <= 2^26 / 64
    return hip_result(idb::launch_aux_stats(c.args.prob_part, c.args.cnt_part, (int)tiles, T, E, alpha, counts, f, P,
                                            loss, out_maxvio_minvio, c.aux_partial, c.ticket, stream),
                      "auxiliary-loss statistics launch");
}

idb_status idb_controller_update_layers(const int32_t* counts, int32_t L, const idb_controller_cfg* cfg,
                                        const idb_controller_state* state, double* out_stats, double* out_diag,
                                        hipStream_t stream) {
    if (!counts) return fail(IDB_ERR_INVALID_ARG, "null pointer");
    if (L < 1 || L > 65535) return fail(IDB_ERR_INVALID_ARG, "L=%d out of [1, 65535]", L);
    idb_status st = check_controller(cfg, state, out_stats);
    if (st != IDB_OK) return st;
    if (!aligned(counts, 4) || (out_diag && !aligned(out_diag, 8))) return fail(IDB_ERR_INVALID_ARG, "misaligned buffer");
    return hip_result(idb::launch_controller_layers(counts, L, cfg->E, cfg->Ki, cfg->Kd,
                                                    cfg->integral_mode == IDB_INTEGRAL_SIGN, cfg->center, state->bias,
                                                    state->e_prev, state->step, state->status, out_stats, out_diag,
                                                    stream),
                      "controller layers launch");
}

size_t idb_routing_entropy_workspace_bytes(void) { return (size_t)idb::kEntropyBlocks * 2 * sizeof(double); }

idb_status idb_routing_entropy(const float* gate_w, int64_t T, int32_t K, const float* scores, const float* bias,
                               int32_t E, void* workspace, size_t workspace_bytes, double* out, hipStream_t stream) {
    if (!gate_w || !out || !workspace) return fail(IDB_ERR_INVALID_ARG, "null pointer");
    if (T < 1 || T > kMaxTokens) return fail(IDB_ERR_INVALID_ARG, "T=%lld out of [1, 2^26]", (long long)T);
    if (K < 1 || K > kMaxKGpu) return fail(IDB_ERR_INVALID_ARG, "K=%d out of [1, %d]", K, kMaxKGpu);
    if (scores && (!bias || E < 1 || E > kMaxExperts))
        return fail(IDB_ERR_INVALID_ARG, "scores need a bias and 1 <= E <= %d", kMaxExperts);
    if (workspace_bytes < idb_routing_entropy_workspace_bytes())
        return fail(IDB_ERR_INVALID_ARG, "workspace of %zu bytes needed", idb_routing_entropy_workspace_bytes());
    if (!aligned(gate_w, 4) || !aligned(out, 8) || !aligned(workspace, 8) || (scores && !aligned(scores, 4)) ||
        (bias && !aligned(bias, 4)))
        return fail(IDB_ERR_INVALID_ARG, "misaligned buffer");
    return hip_result(idb::launch_routing_entropy(gate_w, T, K, scores, bias, E, 0, static_cast<double*>(workspace),
                                                  out, stream),
                      "routing entropy launch");
}

idb_status idb_routing_entropy_softmax(const float* gate_w, int64_t T, int32_t K, const float* logits, int32_t E,
                                       void* workspace, size_t workspace_bytes, double* out, hipStream_t stream) {
    if (!gate_w || !logits || !out || !workspace) return fail(IDB_ERR_INVALID_ARG, "null pointer");
    if (T < 1 || T > kMaxTokens) return fail(IDB_ERR_INVALID_ARG, "T=%lld out of [1, 2^26]", (long long)T);
    if (K < 1 || K > kMaxKGpu) return fail(IDB_ERR_INVALID_ARG, "K=%d out of [1, %d]", K, kMaxKGpu);
    if (E < 1 || E > kMaxExperts) return fail(IDB_ERR_INVALID_ARG, "E=%d out of [1, %d]", E, kMaxExperts);
    if (workspace_bytes < idb_routing_entropy_workspace_bytes())
        return fail(IDB_ERR_INVALID_ARG, "workspace of %zu bytes needed", idb_routing_entropy_workspace_bytes());
    if (!aligned(gate_w, 4) || !aligned(out, 8) || !aligned(workspace, 8) || !aligned(logits, 4))
        return fail(IDB_ERR_INVALID_ARG, "misaligned buffer");
    return hip_result(idb::launch_routing_entropy(gate_w, T, K, logits, nullptr, E, 1,
                                                  static_cast<double*>(workspace), out, stream),
                      "routing entropy launch");
}

idb_status idb_load_stats(const int32_t* counts, int32_t E, double* out_maxvio_minvio, hipStream_t stream) {
    if (!counts || !out_maxvio_minvio) return fail(IDB_ERR_INVALID_ARG, "null pointer");
    if (E < 1 || E > (1 << 20)) return fail(IDB_ERR_INVALID_ARG, "E=%d out of [1, 2^20]", E);
    if (!aligned(counts, 4) || !aligned(out_maxvio_minvio, 8)) return fail(IDB_ERR_INVALID_ARG, "misaligned buffer");
    return hip_result(idb::launch_load_stats(counts, E, out_maxvio_minvio, stream), "load stats launch");
}

const char* idb_status_string(idb_status s) {
    switch (s) {
        case IDB_OK: return "ok";
        case IDB_ERR_INVALID_ARG: return "invalid argument";
        case IDB_ERR_UNSUPPORTED: return "unsupported shape or option";
        case IDB_ERR_EMPTY_BATCH: return "empty batch: every count is zero";
        case IDB_ERR_HIP: return "HIP launch failure";
        default: return "unknown status";
    }
}

const char* idb_last_error(void) { return g_last_error; }

}  // extern "C"
