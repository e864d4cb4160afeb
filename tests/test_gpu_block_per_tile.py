"""Decode of short calls by a block of four wavefronts per tile: all query groups, row lengths whose words end in every place of a
section, sequence ends inside the sixteen tokens of a wavefront, empty sequences, many sequences in a tile, appended rows around the 64
of a block, the most tiles the rule takes.  Against the CPU oracle, tolerance as for plain decode, and against the same call with a given
number of splits, which blocks of four tiles take: neither's largest error is more than a few times the other's."""
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
    tiles_of, form_of = (spark.CALL_DECODE_TAIL_TILES, spark.CALL_DECODE_TAIL) if cap else (spark.CALL_DECODE_TILES, spark.CALL_DECODE)
    assert spark.call_form(desc, tiles_of) == 1
    by_four = make_desc(w, layout, pack, n_splits=(max(w.seqlens) + 255) // 256)
    by_four.tail_capacity = cap
    assert spark.call_form(by_four, tiles_of) == 0 and spark.call_form(by_four, form_of) == 1
    cu = torch.from_numpy(np.asarray(t.cu, np.int32)).cuda()
    k, v = (x if layout == "HND" else np.ascontiguousarray(x.transpose(1, 0, 2)) for x in (t.k, t.v))
    k, v, qwin, q = (to_dev(x) for x in (k, v, t.qwin, t.q))
    packed = torch.empty(spark.packed_bytes(desc), dtype=torch.uint8, device="cuda")
    spark.prune(desc, k, qwin, cu, packed)
    _, _, a32 = oracle.window_stat(t.qwin, w.n_kv_heads)
    pr = oracle.prune(t.k, t.layout, a32, t.cu, w.keep)
    pr = oracle.quant_int8(pr) if pack == spark.PACK_INT8 else pr
    if cap:
        rng = np.random.default_rng(w.batch)
        tk, tv = (wl.f32_to_bf16_bits(rng.standard_normal((w.batch, cap, w.n_kv_heads, 128)).astype(np.float32)) for _ in range(2))
        tl = np.asarray(tail_len, np.int32)
        ref = oracle.decode_literal_tail(t.q, pr, t.v, t.layout, t.cu, tk, tv, tl)
        tk, tv, tl = to_dev(tk), to_dev(tv), torch.from_numpy(tl).cuda()
    else:
        ref = oracle.decode_literal(t.q, pr, t.v, t.layout, t.cu)
    errs = []
    for d in (desc, by_four):
        ws = spark.new_decode_workspace(d)
        for _ in range(2):
            out = torch.full((w.batch, w.n_q_heads, 128), float("nan"), dtype=torch.float32, device="cuda")
            if cap:
                spark.decode_attn_tail(d, q, packed, v, cu, tk, tv, tl, out, ws)
            else:
                spark.decode_attn(d, q, packed, v, cu, out, ws)
            err = np.abs(out.cpu().numpy().astype(np.float64) - ref)
            assert err.max() <= 1e-2 and err.mean() <= 1e-3, (err.max(), err.mean())
        errs.append(err.max())
    print(f"{w.name}: max|err| block per tile {errs[0]:.2e}, four tiles a block {errs[1]:.2e}")
    assert errs[0] <= 4.0 * errs[1] + 2.0 ** -24 * np.abs(ref).max()


@pytest.mark.parametrize("pack", [spark.PACK_BF16, spark.PACK_INT8])
@pytest.mark.parametrize("G,keep", [(G, keep) for G in (1, 2, 4) for keep in (1, 26, 27, 30, 33, 38, 49, 64)])
def test_row_lengths(G, keep, pack):
    if G == 1 and keep == 26 and pack == spark.PACK_INT8:
        keep = 25                                # (never those)
    # (26 and 38 kept channels, four query heads: twenty tiles at most)
    seqlens = (1, 17, 1180) if G == 4 and keep in (26, 38) else (1, 500, 0, 15, 733, 391)
    _check(wl.small(name=f"tile{keep}_{G}", batch=len(seqlens), n_q_heads=2 * G, n_kv_heads=2, keep=keep, seqlens=seqlens, seed=800 + keep + G), pack)


@pytest.mark.parametrize("pack", [spark.PACK_BF16, spark.PACK_INT8])
def test_eight_query_heads(pack):
    _check(wl.small(name="tile8", batch=3, n_q_heads=64, n_kv_heads=8, keep=64, seqlens=(500, 1, 777), seed=810), pack, layout="NHD")


# (from 200 or 240 tokens a sequence on average, or fewer; the most tiles, and the most blocks, that each group takes)
@pytest.mark.parametrize("G,hkv,keep,seqlens", [(1, 8, 64, (2048,)), (1, 2, 64, (6144,)), (2, 8, 64, (2048,)), (2, 4, 64, (4096,)), (4, 8, 64, (2048,)), (4, 1, 64, (200,)), (4, 1, 48, (63, 1)), (2, 3, 40, (1,)), (1, 2, 48, (1,) * 40 + (0,) * 3 + (16, 17, 48, 49)),
                                                (4, 8, 33, (2304,)), (2, 8, 33, (3000, 1060)), (1, 11, 33, (64 * 53, 576)), (8, 8, 64, (1535,)), (2, 3, 64, (241,)),
                                                (4, 2, 64, (65, 0, 0, 927)), (1, 2, 33, (1,) * 15 + (0,) * 3 + (16, 17, 48, 5300))])
def test_sequence_lengths(G, hkv, keep, seqlens):
    _check(wl.small(name=f"tilelen{len(seqlens)}_{G}", batch=len(seqlens), n_q_heads=G * hkv, n_kv_heads=hkv, keep=keep, seqlens=seqlens, seed=820 + G))


@pytest.mark.parametrize("pack", [spark.PACK_BF16, spark.PACK_INT8])
@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_appended_rows(G, pack):
    lens = (0, 1, 63, 64, 65, 200)
    _check(wl.small(name=f"tiletail{G}", batch=6, n_q_heads=2 * G, n_kv_heads=2, keep=64 if G == 8 else 32, seqlens=(5, 0, 300, 64, 17, 600), seed=830 + G), pack, cap=200, tail_len=lens)


@pytest.mark.parametrize("G,keep", [(4, 33), (8, 64)])
def test_only_appended_rows(G, keep):
    _check(wl.small(name=f"tiletail0_{G}", batch=3, n_q_heads=2 * G, n_kv_heads=2, keep=keep, seqlens=(0, 40, 0), seed=840), cap=70, tail_len=(70, 0, 0))


def test_many_sequences_in_a_tile_with_appended_rows():
    _check(wl.small(name="tiletailmany", batch=47, n_q_heads=4, n_kv_heads=2, keep=64, seqlens=(1,) * 40 + (0,) * 3 + (16, 17, 48, 49), seed=850), cap=20, tail_len=(20, 0, 7, 1, 16) * 9 + (17, 20))


def test_the_room_for_a_partial_per_tile_is_not_demanded():
    """A workspace that has room for the partials of four tiles each is accepted; blocks of four tiles then take the call."""
    w = wl.small(name="tileroom", batch=2, n_q_heads=16, n_kv_heads=2, keep=64, seqlens=(700, 520), seed=860)
    t = wl.generate(w)
    desc = make_desc(w)
    assert spark.call_form(desc, spark.CALL_DECODE_TILES) == 1
    whole = spark.decode_workspace_bytes(desc)
    # (chunks: at most (20 tiles + 2 * 2) // 4 + 2 + 1 of them, and a slot for appended rows each)
    least = ((24 // 4 + 3) * 16 + 2 * 16) * 130 * 4 + 4 * 256
    assert least < whole * 2 // 3
    k, v, qwin, q, cu = (to_dev(x) for x in (t.k, t.v, t.qwin, t.q, np.asarray(t.cu, np.int32)))
    packed = torch.empty(spark.packed_bytes(desc), dtype=torch.uint8, device="cuda")
    spark.prune(desc, k, qwin, cu, packed)
    _, _, a32 = oracle.window_stat(t.qwin, 2)
    ref = oracle.decode_literal(t.q, oracle.prune(t.k, t.layout, a32, t.cu, w.keep), t.v, t.layout, t.cu)
    ws = spark.new_decode_workspace(desc)
    outs = []
    for room in (ws, ws[:least // ws.element_size()].clone()):
        out = torch.full((2, 16, 128), float("nan"), dtype=torch.float32, device="cuda")
        spark.decode_attn(desc, q, packed, v, cu, out, room)
        outs.append(out.cpu().numpy())
        assert np.abs(outs[-1] - ref).max() <= 1e-2
    # (a probability is multiplied in two bf16 parts, to 2^-17 of itself at worst, and the probabilities of a row sum to one: each
    #  form is within 2^-17 of the largest value, besides float32 sums)
    assert np.abs(outs[0] - outs[1]).max() <= 2.0 ** -16 * np.abs(wl.bf16_bits_to_f32(t.v)).max()
