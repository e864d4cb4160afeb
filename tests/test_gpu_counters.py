"""Arrival counters of the decode calls, which lie closer together the more (batch, KV head) pairs there are: one workspace, prepared
once, serves calls that cut the same pairs in different ways, one after the other, with the results of fresh workspaces; pairs at
every distance between counters."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
import paper_2508_15212_amd as spark
from tests.gpu_util import make_desc, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,hkv,tokens", [(1, 1, 3000), (2, 8, 700), (3, 6, 500), (11, 3, 333), (8, 8, 300), (13, 5, 200), (43, 3, 150), (37, 8, 90)])
def test_one_workspace_for_all_cuts(batch, hkv, tokens):
    rng = np.random.default_rng(batch)
    lens = tuple(int(x) for x in rng.integers(0, 2 * tokens, size=batch))
    w = wl.small(name=f"counters{batch}x{hkv}", batch=batch, n_q_heads=2 * hkv, n_kv_heads=hkv, keep=26, seqlens=lens, seed=700 + batch)
    t = wl.generate(w)
    cu = torch.from_numpy(np.asarray(t.cu, np.int32)).cuda()
    k, v, qwin, q = (to_dev(x) for x in (t.k, t.v, t.qwin, t.q))
    descs = [make_desc(w, n_splits=n) for n in (0, 1, 5, -1)]
    packed = torch.empty(spark.packed_bytes(descs[0]), dtype=torch.uint8, device="cuda")
    spark.prune(descs[0], k, qwin, cu, packed)
    largest = max(descs, key=spark.decode_workspace_bytes)
    shared = spark.new_decode_workspace(largest)
    _, _, a32 = oracle.window_stat(t.qwin, hkv)
    ref = oracle.decode_literal(t.q, oracle.prune(t.k, t.layout, a32, t.cu, w.keep), t.v, t.layout, t.cu)
    for turn in range(3):
        for desc in descs:
            outs = [torch.full((batch, 2 * hkv, 128), float("nan"), dtype=torch.float32, device="cuda") for _ in range(2)]
            spark.decode_attn(desc, q, packed, v, cu, outs[0], shared)
            spark.decode_attn(desc, q, packed, v, cu, outs[1], spark.new_decode_workspace(desc))
            assert torch.equal(outs[0], outs[1]), (turn, desc.n_splits)
            err = np.abs(outs[0].cpu().numpy().astype(np.float64) - ref)
            assert err.max() <= 1e-2 and err.mean() <= 1e-3


@pytest.mark.parametrize("batch,hkv,G,n_splits", [(1, 1, 1, 0), (1, 1, 1, 3), (2, 2, 1, 7), (3, 2, 2, 4), (4, 8, 4, 5), (2, 1, 8, 2), (64, 8, 1, 2)])
def test_a_workspace_with_room_for_counters_side_by_side_only(batch, hkv, G, n_splits):
    """Counters further apart take up to 2 KB more.  A workspace without that room - the partials, and a word a pair - serves the same
    calls: one after the other, before and after calls of the same workspace whose counters lie apart, and prepared with its own size."""
    lens = tuple(int(x) for x in np.random.default_rng(7 * batch + G).integers(0, 900, size=batch))
    w = wl.small(name=f"narrow{batch}x{hkv}x{G}", batch=batch, n_q_heads=G * hkv, n_kv_heads=hkv, keep=26, seqlens=lens, seed=770 + batch + G)
    t = wl.generate(w)
    k, v, qwin, q, cu = (to_dev(x) for x in (t.k, t.v, t.qwin, t.q, np.asarray(t.cu, np.int32)))
    desc, other = make_desc(w, n_splits=n_splits), make_desc(w, n_splits=1)
    packed = torch.empty(spark.packed_bytes(desc), dtype=torch.uint8, device="cuda")
    spark.prune(desc, k, qwin, cu, packed)
    _, _, a32 = oracle.window_stat(t.qwin, hkv)
    ref = oracle.decode_literal(t.q, oracle.prune(t.k, t.layout, a32, t.cu, w.keep), t.v, t.layout, t.cu)
    tiles = (w.total + 63) // 64
    chunks = batch * n_splits if n_splits else (tiles + 2 * batch) // max(4, -(-tiles * hkv // 512)) + batch + 1
    narrow = (chunks + batch) * G * hkv * 130 * 4 + (batch * hkv * 4 + 255) // 256 * 256
    room = torch.full((max(spark.decode_workspace_bytes(d) for d in (desc, other)) // 4 + 1024,), 0x7F7F7F7F, dtype=torch.int32, device="cuda")
    assert narrow <= spark.decode_workspace_bytes(desc)

    def run(d, words):
        out = torch.full((batch, G * hkv, 128), float("nan"), dtype=torch.float32, device="cuda")
        spark.decode_attn(d, q, packed, v, cu, out, room[:words])
        return out

    spark.decode_workspace_init(desc, room[:narrow // 4])
    outs = []
    for _ in range(3):
        outs += [run(desc, narrow // 4), run(desc, narrow // 4), run(desc, room.numel()), run(other, room.numel())]
    for i, out in enumerate(outs):
        err = np.abs(out.cpu().numpy().astype(np.float64) - ref)
        assert err.max() <= 1e-2 and err.mean() <= 1e-3, (i, err.max())
        # (with all the room a short call takes a block per tile: other last bits)
        if i % 4 < (2 if spark.call_form(desc, spark.CALL_DECODE_TILES) == 1 else 3):
            assert torch.equal(out, outs[0]), i
    with pytest.raises(spark.SparkError):
        run(desc, narrow // 4 - 1)
