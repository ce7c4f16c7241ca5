"""The automatic choice over batch sizes: tilings of 64 and 128 tokens per
workgroup give a token the same bits (scores, selection, gate weights), so its
outputs do not depend on the batch it is routed in.

The comparison is exact: these tilings sum each score over k in the same order
with the same MFMA shape, and the selection is defined bit for bit given the
scores.
"""
import numpy as np
import pytest

from paper_2609_39137_amd import binding as B
from paper_2609_39137_amd import synth
from tests.test_gpu_router import check_invariants, gpu_select, run_router

pytestmark = pytest.mark.gpu


def equal(got, ref):
    for a, g in zip(ref, got):
        np.testing.assert_array_equal(a.view(np.uint32), g.view(np.uint32))


# (variant, the tiling it shares its accumulation order with); one token, the
# edges of a 64-token tile, several tiles; padded and full expert slices; K up
# to the largest, where lists overflow and the slice merge ranks 8 lists
@pytest.mark.parametrize("variant,ref", [(8, 3), (9, 3), (10, 6)])
@pytest.mark.parametrize("T,d,E,K", [(1, 64, 32, 32), (63, 128, 768, 10), (64, 320, 768, 16), (65, 192, 800, 5),
                                     (513, 256, 1024, 32), (200, 64, 256, 1)])
def test_tilings_of_one_order_agree(variant, ref, T, d, E, K):
    x, W = synth.normal_router_inputs(T, d, E, seed=T + E, w_std=0.05)
    b = synth.bias(E, "small", seed=K)
    want = run_router(x, W, b, K, variant=ref)
    got = run_router(x, W, b, K, variant=variant)
    equal(got, want)
    check_invariants(*got[:3], T, E, K)


def resolved(T, E):
    return B.idb_router_variant_info(T, 256, E, 8, B.IDB_DTYPE_BF16, 0)["variant"]


def test_automatic_tiling_by_batch_size():
    # 64-token tiles while they fit one round of the 256 CUs
    assert resolved(8192, 768) == 10 and resolved(8193, 768) == 6
    assert resolved(16384, 384) == 10 and resolved(16385, 384) == 6
    assert resolved(16384, 256) == 9 and resolved(16385, 256) == 8
    assert resolved(4096, 1024) == 9 and resolved(4097, 1024) == 8
    assert resolved(1, 128) == 4


# the last batch on 64-token tiles, the first on 128-token ones: every token
# they share has the same outputs
@pytest.mark.parametrize("T,E,K", [(8192, 768, 10), (4096, 1024, 16), (16384, 256, 8)])
def test_a_token_s_outputs_do_not_depend_on_its_batch(T, E, K):
    x, W = synth.normal_router_inputs(T + 1, 64, E, seed=E, w_std=0.05)
    b = synth.bias(E, "small", seed=2)
    small, large = run_router(np.ascontiguousarray(x[:T]), W, b, K), run_router(x, W, b, K)
    for i in (0, 1, 3):
        np.testing.assert_array_equal(small[i].view(np.uint32), large[i][:T].view(np.uint32))
    si, sw, sc = gpu_select(large[3], b, K)
    equal(large[:3], (si, sw, sc))
