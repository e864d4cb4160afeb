"""The top-p pruning call in one launch and in three: sizes on both sides of the rule that chooses, against the CPU oracle,
and the same buffer used for one call after another (the directory is counted and summed in place)."""
import numpy as np
import pytest
import torch

import workloads as wl
import paper_2508_15212_amd as spark
from tests.gpu_util import make_desc, to_dev
from tests.test_gpu_topp import _run

pytestmark = pytest.mark.gpu


# (KV heads, tokens): one launch up to 256 tiles over all heads, 112 of each, and from 2048 on with four heads or more
@pytest.mark.parametrize("hkv,tokens", [(1, 1), (1, 112 * 64), (1, 113 * 64), (4, 64 * 64 - 9), (1, 256 * 64), (1, 256 * 64 + 1), (8, 32 * 64 - 5), (8, 33 * 64), (4, 511 * 64), (4, 512 * 64 - 1),
                                        (3, 683 * 64), (5, 410 * 64 + 17)])
def test_both_sides_of_the_rule(hkv, tokens):
    tiles = (tokens + 63) // 64
    one = hkv * tiles <= 256 and tiles <= 112 or hkv * tiles >= 2048 and hkv >= 4
    w = wl.small(name=f"topp{hkv}x{tokens}", batch=2, n_q_heads=hkv, n_kv_heads=hkv, seqlens=(tokens - tokens // 3, tokens // 3), seed=351 + hkv)
    assert spark.call_form(make_desc(w), spark.CALL_PRUNE_TOPP) == (1 if one else 3)
    _run(w, wl.generate(w), p_bp=9500, decode=False)


@pytest.mark.parametrize("hkv,tokens", [(2560, 64), (4100, 40), (700, 200)])
def test_more_heads_than_the_chip_holds_blocks(hkv, tokens):
    """No block may wait for one that has not started: 2304 blocks or fewer are resident at once."""
    w = wl.small(name=f"toppheads{hkv}", batch=1, n_q_heads=hkv, n_kv_heads=hkv, seqlens=(tokens,), seed=371)
    assert spark.call_form(make_desc(w), spark.CALL_PRUNE_TOPP) == 1
    _run(w, wl.generate(w), p_bp=9500, decode=False)


@pytest.mark.parametrize("hkv,tokens", [(2, 3000), (8, 16500)])
def test_a_buffer_used_again_holds_the_last_call(hkv, tokens):
    ws = [wl.small(name=f"again{s}", batch=1, n_q_heads=hkv, n_kv_heads=hkv, seqlens=(tokens,), seed=s) for s in (361, 362)]
    ts = [wl.generate(w) for w in ws]
    desc = make_desc(ws[0], "HND")
    cu = torch.tensor([0, tokens], dtype=torch.int32, device="cuda")
    dev = [(to_dev(t.k), to_dev(t.qwin)) for t in ts]

    def call(i, p, packed):
        spark.prune_topp(desc, dev[i][0], dev[i][1], cu, p, packed)
        return packed

    fresh = [call(0, 9900, torch.zeros(spark.packed_topp_bytes(desc), dtype=torch.uint8, device="cuda")).clone(),
             call(1, 3000, torch.zeros(spark.packed_topp_bytes(desc), dtype=torch.uint8, device="cuda")).clone()]
    n_tiles = (tokens + 63) // 64
    mask = torch.empty((2, tokens, hkv, 4), dtype=torch.int32, device="cuda")
    vals = torch.empty((2, tokens, hkv, 128), dtype=torch.int16, device="cuda")
    packed = torch.zeros_like(fresh[0])
    for step in range(12):
        i = step % 2
        call(i, (9900, 3000)[i], packed)
        for n, p in enumerate((packed, fresh[i])):
            spark.unpack_topp(desc, p, mask[n], None, vals[n], None, None)
        assert torch.equal(mask[0], mask[1]) and torch.equal(vals[0], vals[1]), f"call {step}"
    assert n_tiles > 0 and np.all(mask[0].cpu().numpy().any(axis=-1))
