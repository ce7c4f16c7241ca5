"""Workspace sizes of the automatic choices over batch sizes (host only): what
a caller allocates, that the plain choice asks for the fused tiling's part alone
(and so keeps to it), and which calls take the scored path."""
import ctypes

import pytest

from paper_2609_39137_amd import binding as B

A16 = ctypes.c_void_p(1 << 12)  # an aligned address that no check dereferences


def fused_bytes(T, slices, K):
    return 3 * ((T * slices * K * 4 + 255) // 256 * 256) + 256 if slices > 1 else 0


def scored_bytes(T, E):
    return (T * E * 4 + 255) // 256 * 256 + 256


# (T, d, E, K, dtype, slices, scored, packs): both sides of each line of the
# choice; `scored` for either weight layout, since the query has none
@pytest.mark.parametrize("T,d,E,K,dtype,slices,scored,packs", [
    (32, 2048, 768, 10, 0, 2, True, False),
    (2560, 2048, 768, 10, 0, 2, True, True),
    (8192, 2048, 768, 10, 0, 2, True, True),      # row-major only
    (8193, 2048, 768, 10, 0, 2, False, False),
    (16384, 2048, 768, 12, 0, 2, False, False),
    (16384, 2048, 768, 13, 0, 2, True, True),
    (65536, 2048, 1024, 21, 0, 4, True, True),
    (65537, 2048, 1024, 21, 0, 4, False, False),  # above 256 MB of scores
    (777, 4096, 256, 8, 0, 1, True, False),
    (24577, 4096, 256, 8, 0, 1, False, False),
    (2730, 512, 768, 10, 0, 2, True, True),       # row-major only, smaller hidden sizes
    (2731, 512, 768, 10, 0, 2, False, False),
    (1280, 256, 768, 10, 0, 2, True, True),
    (1281, 256, 768, 10, 0, 2, False, False),
    (8192, 1024, 384, 13, 0, 1, True, True),      # K > 12, one slice
    (8193, 1024, 384, 13, 0, 1, False, False),
    (8193, 1024, 384, 14, 0, 1, True, True),
    (8193, 2048, 384, 14, 0, 1, False, False),
    (8193, 2048, 384, 15, 0, 1, True, True),
    (12288, 64, 256, 20, 0, 1, True, True),
    (12289, 64, 256, 20, 0, 1, False, False),
    (12289, 64, 256, 21, 0, 1, True, True),
    (43690, 1024, 768, 13, 0, 2, True, True),     # several slices
    (43691, 1024, 768, 13, 0, 2, False, False),
    (43691, 512, 768, 13, 0, 2, True, True),
    (43691, 1024, 768, 14, 0, 2, True, True),
    (12288, 64, 1024, 20, 0, 4, True, True),
    (12289, 64, 1024, 20, 0, 4, False, False),
    (16384, 512, 128, 8, 0, 1, True, True),       # 128-expert tiles
    (16385, 512, 128, 8, 0, 1, False, False),
    (14336, 64, 128, 8, 0, 1, True, True),
    (14337, 64, 128, 8, 0, 1, False, False),
    (20480, 512, 64, 8, 0, 1, True, True),
    (20481, 512, 64, 8, 0, 1, False, False),
    (3510, 64, 896, 1, 0, 7, True, True),
    (3511, 64, 896, 1, 0, 7, False, False),
    (7021, 64, 896, 2, 0, 7, True, True),
    (7022, 64, 896, 2, 0, 7, False, False),
    (32768, 256, 64, 4, 1, 1, True, False),       # fp32 is never packed on the way
    (32769, 256, 64, 4, 1, 1, False, False),
    (24576, 64, 64, 4, 1, 1, True, False),
    (24577, 64, 64, 4, 1, 1, False, False),
])
def test_workspace_covers_the_path_of_either_layout(T, d, E, K, dtype, slices, scored, packs):
    assert B.idb_router_variant_info(T, d, E, K, dtype, 0)["slices"] == slices
    fused = fused_bytes(T, slices, K)
    want = max(fused, scored_bytes(T, E) + (E * d * 2 if packs else 0)) if scored else fused
    assert B.idb_router_workspace_bytes(T, d, E, K, dtype, B.IDB_ROUTER_AUTO_SCORES) == want
    # the plain automatic choice and a forced variant use the fused tiling's part only
    v = B.idb_router_variant_info(T, d, E, K, dtype, 0)["variant"]
    assert B.idb_router_workspace_bytes(T, d, E, K, dtype, 0) == fused
    assert B.idb_router_workspace_bytes(T, d, E, K, dtype, v) == fused
    # the path: with that workspace some layout takes it; with one too small
    # for the scores, or without the choice that owns the workspace, none does
    layouts = (B.IDB_WEIGHT_ROW_MAJOR, B.IDB_WEIGHT_PACKED)
    assert any(B.idb_router_uses_scores(T, d, E, K, dtype, w, want) for w in layouts) == scored
    for w in layouts:
        assert not B.idb_router_uses_scores(T, d, E, K, dtype, w, scored_bytes(T, E) - 1)
        assert not B.idb_router_uses_scores(T, d, E, K, dtype, w, 1 << 40, 0)
        assert not B.idb_router_uses_scores(T, d, E, K, dtype, w, 1 << 40, v)


def test_only_whole_router_calls_accept_the_workspace_owning_choice():
    L, v = B.lib(), B.IDB_ROUTER_AUTO_SCORES
    args = [A16, A16, 0, 0, A16, 300, 128, 768, 10, A16, A16, A16, 0, None, A16, 1 << 30, v, None]
    assert L.idb_router_score_select(*args) == B.IDB_ERR_INVALID_ARG
    assert L.idb_router_merge(300, 128, 768, 10, 0, A16, A16, A16, A16, 1 << 30, v, None) == B.IDB_ERR_INVALID_ARG
    assert B.idb_qb_router_workspace_bytes(300, 128, 768, 10, 0, v) == 0
    assert B.idb_aux_router_workspace_bytes(300, 128, 768, 10, 0, v) == 0
    args[14], args[15] = A16, fused_bytes(300, 2, 10) - 1  # as variant 0: the fused part is the least
    assert L.idb_router_forward(*args) == B.IDB_ERR_INVALID_ARG
    assert b"workspace" in L.idb_last_error()


def test_less_than_the_fused_workspace_is_refused():
    # (that the query's size is enough is seen on a GPU, where RouterStep
    # allocates just that: no check comes after it)
    L = B.lib()
    T, E, K = 300, 768, 10
    need = fused_bytes(T, 2, K)
    fwd = [A16, A16, 0, 0, A16, T, 128, E, K, A16, A16, A16, 0, None]
    for ws, n in ((A16, need - 1), (None, need)):
        for v in (0, B.IDB_ROUTER_AUTO_SCORES):
            assert L.idb_router_forward(*fwd, ws, n, v, None) == B.IDB_ERR_INVALID_ARG
            assert b"workspace" in L.idb_last_error()
        assert L.idb_router_merge(T, 128, E, K, 0, A16, A16, A16, ws, n, 0, None) == B.IDB_ERR_INVALID_ARG
        assert b"workspace" in L.idb_last_error()
