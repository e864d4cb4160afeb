"""Short pruning calls, whose blocks compute the channel weights of their tile's sequences themselves: weights, masks, kept
entries and means against the oracle and, bit for bit, against the launch that takes its weights from memory (which a window
that is only 2-byte aligned gets).  Sequences that end inside a tile, many in one tile, empty ones, window lengths around the
eight and 32 rows of a request, all query-group sizes."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
import paper_2508_15212_amd as spark
from tests.gpu_util import make_desc, to_dev

pytestmark = pytest.mark.gpu


def _packed(desc, t, shift):
    buf = torch.zeros(t.qwin.size + 8, dtype=torch.int16, device="cuda")
    qwin = buf[shift:shift + t.qwin.size]
    qwin.copy_(to_dev(t.qwin).reshape(-1))
    packed = torch.zeros(spark.packed_bytes(desc), dtype=torch.uint8, device="cuda")
    spark.prune(desc, to_dev(t.k), qwin, torch.from_numpy(np.asarray(t.cu, np.int32)).cuda(), packed)
    return packed


@pytest.mark.parametrize("pack,stats", [(spark.PACK_BF16, 0), (spark.PACK_INT8, 0), (spark.PACK_BF16, 1), (spark.PACK_INT8, 1)])
@pytest.mark.parametrize("G,window", [(1, 1), (2, 7), (4, 32), (8, 41), (2, 64)])
@pytest.mark.parametrize("seqlens", [(1000,), (300, 0, 261, 700), (1, 2, 0, 3, 0, 4000, 1, 5, 0), (1,) * 70 + (20000,)])
def test_weights_in_the_pruning_launch(seqlens, G, window, pack, stats):
    hkv = 1 if len(seqlens) > 50 else 2
    w = wl.small(name=f"win{len(seqlens)}_{G}", batch=len(seqlens), n_q_heads=G * hkv, n_kv_heads=hkv, keep=30, seqlens=seqlens, seed=600 + G)
    w.window = window
    t = wl.generate(w)
    desc = make_desc(w, pack=pack)
    desc.stats = stats
    assert spark.call_form(desc, spark.CALL_PRUNE) == 1
    got, ref = _packed(desc, t, 0), _packed(desc, t, 1)
    assert torch.equal(got, ref)
    if pack == spark.PACK_BF16 and not stats:
        _against_oracle(w, t, desc, got)


def _against_oracle(w, t, desc, packed):
    hkv = w.n_kv_heads
    mask = torch.empty((w.total, hkv, 4), dtype=torch.int32, device="cuda")
    a = torch.empty((w.batch, hkv, 128), dtype=torch.float32, device="cuda")
    spark.unpack(desc, packed, mask, None, None, None, a)
    _, _, a32 = oracle.window_stat(t.qwin, hkv)
    assert np.array_equal(a.cpu().numpy().view(np.uint32), np.asarray(a32, np.float32).reshape(w.batch, hkv, 128).view(np.uint32))
    assert np.array_equal(mask.cpu().numpy().view(np.uint32), oracle.prune(t.k, t.layout, a32, t.cu, w.keep).mask)


# (a block per tile and one per sequence, over the heads: up to 768)
@pytest.mark.parametrize("hkv,tokens,launches", [(1, 767 * 64, 1), (1, 767 * 64 + 1, 2), (8, 95 * 64 - 3, 1), (8, 95 * 64 + 1, 2)])
def test_both_sides_of_the_rule(hkv, tokens, launches):
    w = wl.small(name=f"winrule{hkv}x{tokens}", batch=1, n_q_heads=hkv, n_kv_heads=hkv, keep=30, seqlens=(tokens,), seed=620 + hkv)
    t = wl.generate(w)
    desc = make_desc(w)
    assert spark.call_form(desc, spark.CALL_PRUNE) == launches
    got = _packed(desc, t, 0)
    assert torch.equal(got, _packed(desc, t, 1))
    _against_oracle(w, t, desc, got)
