"""Decode of short calls by a block of four wavefronts per tile: all query groups, row lengths whose words end in every place of a
section, sequence ends inside the sixteen tokens of a wavefront, empty sequences, many sequences in a tile, appended rows around the 64
of a block, the most tiles the rule takes.  Against the CPU oracle, tolerance as for plain decode, and against the same call with a workspace
that only has room for the partials of four tiles each (which the library accepts): neither's largest error is more than a few times
the other's."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
import paper_2508_15212_amd as spark
from tests.gpu_util import make_desc, to_dev

pytestmark = pytest.mark.gpu


def _check(w, pack=spark.PACK_BF16, layout="HND", cap=0, tail_len=()):
    t = wl.generate(w)
    desc = make_desc(w, layout, pack)
    desc.tail_capacity = cap
    assert spark.call_form(desc, spark.CALL_DECODE_TAIL if cap else spark.CALL_DECODE) == 1
    cu = torch.from_numpy(np.asarray(t.cu, np.int32)).cuda()
    k, v = (x if layout == "HND" else np.ascontiguousarray(x.transpose(1, 0, 2)) for x in (t.k, t.v))
    k, v, qwin, q = (to_dev(x) for x in (k, v, t.qwin, t.q))
    packed = torch.empty(spark.packed_bytes(desc), dtype=torch.uint8, device="cuda")
    spark.prune(desc, k, qwin, cu, packed)
    _, _, a32 = oracle.window_stat(t.qwin, w.n_kv_heads)
    pr = oracle.prune(t.k, t.layout, a32, t.cu, w.keep)
    pr = oracle.quant_int8(pr) if pack == spark.PACK_INT8 else pr
    whole = spark.new_decode_workspace(desc)
    # partials of four tiles each: (tiles + 2 batch) / 4 + batch chunks, the appended rows' by 256, and the counters
    tiles = (w.total + 63) // 64
    slots = (tiles + 2 * w.batch) // 4 + w.batch + 1 + w.batch * max(1, (cap + 255) // 256)
    least = slots * w.n_q_heads * 130 * 4 + 2048
    bytes_of = lambda ws: ws.numel() * ws.element_size()
    assert bytes_of(whole) > least or tiles < 12, "the call does not take a block per tile"     # (few tiles: the sizes cross)
    if cap:
        rng = np.random.default_rng(w.batch)
        tk, tv = (wl.f32_to_bf16_bits(rng.standard_normal((w.batch, cap, w.n_kv_heads, 128)).astype(np.float32)) for _ in range(2))
        tl = np.asarray(tail_len, np.int32)
        ref = oracle.decode_literal_tail(t.q, pr, t.v, t.layout, t.cu, tk, tv, tl)
        tk, tv, tl = to_dev(tk), to_dev(tv), torch.from_numpy(tl).cuda()
    else:
        ref = oracle.decode_literal(t.q, pr, t.v, t.layout, t.cu)
    errs = []
    for ws in (whole, whole[:least // whole.element_size()].clone()):
        for _ in range(2):
            out = torch.full((w.batch, w.n_q_heads, 128), float("nan"), dtype=torch.float32, device="cuda")
            if cap:
                spark.decode_attn_tail(desc, q, packed, v, cu, tk, tv, tl, out, ws)
            else:
                spark.decode_attn(desc, q, packed, v, cu, out, ws)
            err = np.abs(out.cpu().numpy().astype(np.float64) - ref)
            assert err.max() <= 1e-2 and err.mean() <= 1e-3, (err.max(), err.mean())
        errs.append(err.max())
    print(f"{w.name}: max|err| block per tile {errs[0]:.2e}, four tiles a block {errs[1]:.2e}")
    assert errs[0] <= 4.0 * errs[1] + 2.0 ** -24 * np.abs(ref).max()


@pytest.mark.parametrize("pack", [spark.PACK_BF16, spark.PACK_INT8])
@pytest.mark.parametrize("G", [1, 2, 4])
@pytest.mark.parametrize("keep", [1, 27, 30, 33, 38, 49, 64])
def test_row_lengths(keep, G, pack):
    _check(wl.small(name=f"tile{keep}_{G}", batch=6, n_q_heads=2 * G, n_kv_heads=2, keep=keep, seqlens=(1, 700, 0, 15, 833, 451), seed=800 + keep + G), pack)


def test_eight_query_heads():
    _check(wl.small(name="tile8", batch=3, n_q_heads=64, n_kv_heads=8, keep=64, seqlens=(500, 1, 777), seed=810), layout="NHD")


@pytest.mark.parametrize("G,hkv,seqlens", [(1, 8, (4096,)), (1, 16, (2600,)), (2, 8, (3000,)), (4, 8, (2047,)), (4, 1, (64,)), (4, 1, (63, 1)), (2, 3, (1,)), (4, 2, (65, 0, 0, 127)),
                                           (1, 2, (1,) * 40 + (0,) * 3 + (16, 17, 48, 49))])
def test_sequence_lengths(G, hkv, seqlens):
    _check(wl.small(name=f"tilelen{len(seqlens)}_{G}", batch=len(seqlens), n_q_heads=G * hkv, n_kv_heads=hkv, keep=64, seqlens=seqlens, seed=820 + G))


@pytest.mark.parametrize("G", [1, 2, 4])
def test_appended_rows(G):
    lens = (0, 1, 63, 64, 65, 200)
    _check(wl.small(name=f"tiletail{G}", batch=6, n_q_heads=2 * G, n_kv_heads=2, keep=32, seqlens=(5, 0, 300, 64, 17, 900), seed=830 + G), cap=200, tail_len=lens)


def test_only_appended_rows():
    _check(wl.small(name="tiletail0", batch=3, n_q_heads=8, n_kv_heads=2, keep=33, seqlens=(0, 40, 0), seed=840), cap=70, tail_len=(70, 0, 0))
