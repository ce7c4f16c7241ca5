"""The automatic choice over batch sizes: tilings of 32, 64 and 128 tokens
per workgroup give a token the same bits (scores, selection, gate weights), so its
outputs do not depend on the batch it is routed in.

The comparison is exact: these tilings sum each score over k in the same order
with the same MFMA shape, and the selection is defined bit for bit given the
scores.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_39137_amd import binding as B
from paper_2609_39137_amd import synth
from paper_2609_39137_amd.pipeline import RouterStep
from tests.test_gpu_router import DEV, check_invariants, gpu_select, run_router, to_dev

pytestmark = pytest.mark.gpu


def equal(got, ref):
    for a, g in zip(ref, got):
        np.testing.assert_array_equal(a.view(np.uint32), g.view(np.uint32))


# (variant, the tiling it shares its accumulation order with); one token, the
# edges of a 64-token tile, several tiles; padded and full expert slices; K up
# to the largest, where lists overflow and the slice merge ranks 8 lists
@pytest.mark.parametrize("variant,ref", [(8, 3), (9, 3), (10, 6), (11, 6), (12, 3)])
@pytest.mark.parametrize("T,d,E,K", [(1, 64, 32, 32), (63, 128, 768, 10), (64, 320, 768, 16), (65, 192, 800, 5),
                                     (513, 256, 1024, 32), (200, 64, 256, 1)])
def test_tilings_of_one_order_agree(variant, ref, T, d, E, K):
    x, W = synth.normal_router_inputs(T, d, E, seed=T + E, w_std=0.05)
    b = synth.bias(E, "small", seed=K)
    want = run_router(x, W, b, K, variant=ref)
    got = run_router(x, W, b, K, variant=variant)
    equal(got, want)
    check_invariants(*got[:3], T, E, K)


# the slice merge against the oracle's selection on the kernel's own scores, bit
# for bit: 3 to 8 slices, list lengths that are scanned and that are searched,
# both merge kernels (up to 64 candidates per token and more), and ties that are
# decided by the index across slices
@pytest.mark.parametrize("E,variant", [(640, 3), (1024, 8), (800, 4), (1024, 4)])
@pytest.mark.parametrize("K", [1, 7, 8, 9, 10, 11, 12, 15, 16, 17, 24, 32])
def test_slice_merge_matches_the_oracle(E, variant, K):
    T, d = 150, 64
    x, W = synth.normal_router_inputs(T, d, E, seed=E + K, w_std=0.05)
    for ties in (False, True):
        if ties:
            W[::3] = W[0]
        b = synth.bias(E, "zero" if ties else "small", seed=K)
        idx, w, c, s = run_router(x, W, b, K, variant=variant)
        for got, want in zip((idx, w, c), oracle.select(s, b, K)):
            np.testing.assert_array_equal(got.view(np.uint32), want.view(np.uint32))


def resolved(T, E):
    return B.idb_router_variant_info(T, 256, E, 8, B.IDB_DTYPE_BF16, 0)["variant"]


def test_automatic_tiling_by_batch_size():
    # 64- and, up to 4096 tokens, 32-token tiles while they fit one round of the 256 CUs
    assert resolved(8192, 768) == 10 and resolved(8193, 768) == 6
    assert resolved(16384, 384) == 10 and resolved(16385, 384) == 6
    assert resolved(16384, 256) == 9 and resolved(16385, 256) == 8
    assert resolved(4096, 1024) == 9 and resolved(4097, 1024) == 8
    assert resolved(1, 128) == 4
    assert resolved(4096, 768) == 11 and resolved(4097, 768) == 10
    assert resolved(4096, 256) == 12 and resolved(4097, 256) == 9
    assert resolved(2048, 1024) == 12 and resolved(2049, 1024) == 9


# the last batch on one tile size of the fused tilings and the first on the next:
# every token they share has the same outputs
@pytest.mark.parametrize("T,E,K", [(8192, 768, 10), (4096, 768, 10), (4096, 1024, 16), (16384, 256, 8), (4096, 512, 3)])
def test_a_token_s_outputs_do_not_depend_on_its_batch(T, E, K):
    assert resolved(T, E) != resolved(T + 1, E)
    x, W = synth.normal_router_inputs(T + 1, 64, E, seed=E, w_std=0.05)
    b = synth.bias(E, "small", seed=2)
    small, large = run_router(np.ascontiguousarray(x[:T]), W, b, K), run_router(x, W, b, K)
    for i in (0, 1, 3):
        np.testing.assert_array_equal(small[i].view(np.uint32), large[i][:T].view(np.uint32))
    si, sw, sc = gpu_select(large[3], b, K)
    equal(large[:3], (si, sw, sc))


# the tilings that batches of more than 4096 tokens run, against the oracle on
# integer inputs (exact logits, a zero bias: the selection is decided identically)
@pytest.mark.parametrize("T,E,K,tiling", [(4097, 768, 10, 10), (8193, 736, 4, 6), (4097, 256, 8, 9), (16385, 256, 3, 8),
                                          (4097, 1024, 5, 8), (4100, 512, 8, 9), (4097, 384, 12, 10)])
def test_tilings_of_large_batches_match_the_oracle(T, E, K, tiling):
    x, W = synth.integer_router_inputs(T, 64, E, seed=T + E, dtype="bf16", w_shift=6)
    rs = RouterStep(T, 64, E, K, torch.bfloat16, B.ControllerCfg(E))
    rs.pack(to_dev(W))
    assert rs.info["variant"] == tiling and not rs.uses_scores(packed=True)
    rs.step(to_dev(x))
    ref = oracle.ControllerState(E)
    r_idx, r_w, r_c = oracle.router(x, W, ref.bias, K)
    np.testing.assert_array_equal(rs.idx.cpu().numpy(), r_idx)
    np.testing.assert_array_equal(rs.counts.cpu().numpy(), r_c)
    np.testing.assert_allclose(rs.w.cpu().numpy(), r_w, rtol=2e-5)
    oracle.controller(r_c, ref, rs.cfg.Ki, rs.cfg.Kd)
    np.testing.assert_array_equal(rs.state.bias.cpu().numpy().view(np.uint32), ref.bias.view(np.uint32))
    np.testing.assert_array_equal(rs.stats.cpu().numpy(), oracle.load_stats(r_c))


# the scored path (RouterStep's automatic choice: small batches, large K,
# row-major router matrices) against the fused tiling of the same order, bit for
# bit: scores, selection, counts over two microbatches, and the controller
# update; (T, d, E, K, dtype): both MFMA shapes and fp32, every tile size, part
# tiles, fewer chunks than are prefetched, odd chunk counts, every number of
# selection groups, the sizes of selection workgroups; then expert blocks that
# do not divide E: 32x32 tiles of 64 x 128, 16x16 tiles of 64 x 64, 64 x 128, 64 x 192
# and 128 x 384
SCORED = [(1, 64, 32, 32, "bf16"), (16, 128, 768, 10, "bf16"), (17, 576, 384, 13, "bf16"),
          (257, 64, 768, 16, "bf16"), (1025, 448, 768, 10, "bf16"), (2100, 64, 768, 24, "bf16"),
          (4097, 64, 768, 20, "bf16"), (14500, 64, 768, 17, "bf16"), (33, 64, 64, 4, "bf16"),
          (777, 256, 256, 8, "bf16"), (1500, 192, 1024, 16, "bf16"), (700, 128, 640, 11, "bf16"),
          (4100, 64, 1024, 32, "bf16"), (1200, 64, 512, 3, "bf16"), (31, 32, 64, 4, "f32"), (1000, 288, 128, 21, "f32"),
          (4096, 256, 64, 1, "f32"),
          (7700, 128, 96, 8, "bf16"), (900, 64, 736, 10, "bf16"), (1700, 64, 352, 16, "bf16"), (3500, 64, 352, 13, "bf16"),
          (5100, 64, 352, 14, "bf16"), (14300, 64, 736, 14, "bf16"), (28600, 64, 352, 16, "bf16")]
# a row-major matrix that is packed on the way, where a packed one takes the fused tiling
ROW_MAJOR = [(2000, 448, 512, 8, "bf16"), (8000, 768, 736, 4, "bf16")]


@pytest.mark.parametrize("T,d,E,K,dtype,packed", [(*c, p) for c in SCORED for p in (False, True)] +
                         [(*c, False) for c in ROW_MAJOR])
@pytest.mark.parametrize("ties", [False, True])
def test_scored_path_equals_the_fused_tiling(T, d, E, K, dtype, packed, ties):
    x, W = synth.normal_router_inputs(T, d, E, seed=T + K, dtype=dtype, w_std=0.05)
    if ties:  # equal rows: lists that overflow, ranks decided by the index
        W[: E // 2] = W[0]
    code = B.IDB_DTYPE_BF16 if dtype == "bf16" else B.IDB_DTYPE_F32
    xt, Wt = to_dev(x), to_dev(W)
    fused = B.idb_router_variant_info(T, d, E, K, code, 0)["variant"]
    outs = []
    for variant in (0, fused):
        rs = RouterStep(T, d, E, K, xt.dtype, B.ControllerCfg(E), variant=variant)
        assert rs.uses_scores(packed) == (variant == 0)
        rs.state.bias.copy_(torch.from_numpy(synth.bias(E, "zero" if ties else "small", seed=K)))
        Wa = None if packed else Wt
        if packed:
            rs.pack(Wt)
        dump = torch.full((T, E), -1.0, dtype=torch.float32, device=DEV)
        rs.route(xt, Wa, scores_dump=dump)
        got = [dump.clone(), rs.idx.clone(), rs.w.clone(), rs.counts.clone()]
        rs.step(xt, Wa)
        rs.step(xt, Wa, accumulate=True)
        got += [t.clone() for t in (rs.idx, rs.w, rs.counts, rs.state.bias, rs.state.e_prev, rs.state.step,
                                    rs.state.status, rs.stats)]
        outs.append([t.cpu().numpy() for t in got])
    for a, g in zip(*outs):
        np.testing.assert_array_equal(a.view(np.uint32), g.view(np.uint32))


# one-slice tilings (no workspace of their own) and several slices, both types
@pytest.mark.parametrize("T,d,E,K,dtype", [(300, 128, 256, 8, "bf16"), (1100, 64, 64, 32, "bf16"), (100, 64, 64, 4, "f32"),
                                           (300, 128, 768, 10, "bf16"), (2000, 64, 1024, 24, "bf16")])
def test_variant_0_touches_only_its_part_of_the_workspace(T, d, E, K, dtype):
    # the rest of a pooled scratch may belong to calls on other streams; the
    # choice that owns it all gives the same bits
    x, W = synth.normal_router_inputs(T, d, E, seed=T, dtype=dtype, w_std=0.05)
    code = B.IDB_DTYPE_BF16 if dtype == "bf16" else B.IDB_DTYPE_F32
    bias = torch.from_numpy(synth.bias(E, "small", seed=1)).to(DEV)
    own = B.idb_router_workspace_bytes(T, d, E, K, code, 0)
    size = max(own, T * E * 4 + E * d * 4) + 4096
    outs = []
    for variant in (0, B.IDB_ROUTER_AUTO_SCORES):
        pool = torch.full((size,), 0x5A, dtype=torch.uint8, device=DEV)
        st = B.ControllerState(E, DEV)
        st.bias.copy_(bias)
        idx = torch.empty((T, K), dtype=torch.int32, device=DEV)
        w = torch.empty((T, K), dtype=torch.float32, device=DEV)
        c = torch.empty(E, dtype=torch.int32, device=DEV)
        stats = torch.empty(2, dtype=torch.float64, device=DEV)
        got = []
        B.idb_router_forward(to_dev(x), to_dev(W), bias, K, idx, w, c, workspace=pool, variant=variant)
        got += [t.cpu().numpy() for t in (idx, w, c)]
        B.idb_router_step(to_dev(x), to_dev(W), K, B.ControllerCfg(E), st, idx, w, c, False, stats, pool, variant)
        got += [t.cpu().numpy() for t in (idx, w, c, st.bias, st.e_prev, st.step, stats)]
        outs.append(got)
        untouched = bool((pool[own:] == 0x5A).all())
        scored = B.idb_router_uses_scores(T, d, E, K, code, B.IDB_WEIGHT_ROW_MAJOR, size, variant)
        assert scored == (variant != 0) and untouched == (variant == 0)
    equal(*outs)


def test_a_workspace_sized_for_the_fused_tiling_keeps_it():
    # a caller that sized its workspace by the fused tiling (or passes none to
    # a one-slice tiling) is served as before, with the same outputs
    for T, E, K, ws_bytes in ((300, 768, 10, 3 * (300 * 2 * 10 * 4 + 255) // 256 * 256 + 1024), (300, 256, 8, 0)):
        x, W = synth.normal_router_inputs(T, 128, E, seed=T, w_std=0.05)
        want = run_router(x, W, synth.bias(E, "small", seed=1), K, dump=False)
        assert B.idb_router_workspace_bytes(T, 128, E, K, B.IDB_DTYPE_BF16, B.IDB_ROUTER_AUTO_SCORES) > ws_bytes
        idx = torch.empty((T, K), dtype=torch.int32, device=DEV)
        w = torch.empty((T, K), dtype=torch.float32, device=DEV)
        c = torch.empty(E, dtype=torch.int32, device=DEV)
        ws = torch.empty(ws_bytes, dtype=torch.uint8, device=DEV) if ws_bytes else None
        B.idb_router_forward(to_dev(x), to_dev(W), torch.from_numpy(synth.bias(E, "small", seed=1)).to(DEV), K, idx, w,
                             c, workspace=ws, variant=B.IDB_ROUTER_AUTO_SCORES)
        equal([idx.cpu().numpy(), w.cpu().numpy(), c.cpu().numpy()], want[:3])
