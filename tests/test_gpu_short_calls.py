"""Decode of short calls by blocks of sixteen wavefronts, sixteen tokens a wavefront, four lanes a row: row lengths whose words
end in every place of a section, rows whose kept channels all lie in one mask word, sequence ends inside the sixteen tokens,
empty sequences, chunks of more than one pass, appended rows around the sixteen of a wavefront and the 256 of a block, and the
merge of one partial and of many.  Against the CPU oracle, tolerance as for plain decode; and by the same cache decoded by blocks
of four wavefronts, which compute the same in the same precision: neither's largest error is more than a few times the other's
(the output of a kernel that lost the second part of its probabilities is some 2^8 times further off)."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
import paper_2508_15212_amd as spark
from tests.gpu_util import make_desc, run_gpu_case, to_dev
from tests.test_gpu_tail import _tail_case

pytestmark = pytest.mark.gpu
MAX_ABS, MEAN_ABS = 1e-2, 1e-3


def _check(w, t, pack=spark.PACK_BF16, n_splits=0, layout="HND", form=2):
    desc = make_desc(w, layout, pack, n_splits=n_splits)
    assert spark.call_form(desc, spark.CALL_DECODE) == form
    res = run_gpu_case(w, t, layout=layout, pack=pack, n_splits=n_splits, want_unpack=False)
    _, _, a32 = oracle.window_stat(t.qwin, w.n_kv_heads)
    pr = oracle.prune(t.k, t.layout, a32, t.cu, w.keep)
    pr = oracle.quant_int8(pr) if pack == spark.PACK_INT8 else pr
    ref = oracle.decode_literal(t.q, pr, t.v, t.layout, t.cu)
    err = np.abs(res["out_f32"].astype(np.float64) - ref)
    assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS, (err.max(), err.mean())
    if form == 2:
        # more chunks than there are compute units: blocks of four wavefronts
        desc = make_desc(w, layout, pack, n_splits=256 // w.n_kv_heads // w.batch + 1)
        assert spark.call_form(desc, spark.CALL_DECODE) == 1
        out = torch.empty((w.batch, w.n_q_heads, 128), dtype=torch.float32, device="cuda")
        _, dv, _, dq, dcu = res["dev"]
        spark.decode_attn(desc, dq, res["packed"], dv, dcu, out, spark.new_decode_workspace(desc))
        other = np.abs(out.cpu().numpy().astype(np.float64) - ref)
        print(f"{w.name}: max|err| sixteen wavefronts {err.max():.2e}, four {other.max():.2e}")
        assert err.max() <= 4.0 * other.max() + 2.0 ** -24 * np.abs(ref).max()
    # (half a unit of bf16's last place is 2^-9 of a value at most)
    assert np.abs(res["out_bf16"] - res["out_f32"]).max() <= 2.0 ** -8 * np.abs(res["out_f32"]).max()


# Short rows take these blocks with many tiles a sequence only: one long sequence among short ones
FEW_LONG = dict(batch=3, seqlens=(15, 18433, 0))


@pytest.mark.parametrize("pack", [spark.PACK_BF16, spark.PACK_INT8])
@pytest.mark.parametrize("G,Hkv", [(1, 8), (2, 8), (4, 8), (8, 1)])
@pytest.mark.parametrize("keep", [1, 27, 66, 67, 126, 128])
def test_row_lengths(keep, G, Hkv, pack):
    batch = dict(batch=6, seqlens=(1, 1700, 0, 15, 2033, 451))
    if G < 8 and keep <= (80 if G == 2 else 64):
        batch, Hkv = FEW_LONG, 2
    w = wl.small(name=f"short{keep}_{G}", n_q_heads=G * Hkv, n_kv_heads=Hkv, keep=keep, seed=500 + keep + G, **batch)
    _check(w, wl.generate(w), pack)


@pytest.mark.parametrize("keep", [26, 64, 38])
def test_eight_query_heads_instantiated_lengths(keep):
    w = wl.small(name=f"short8_{keep}", n_q_heads=16, n_kv_heads=2, keep=keep, seed=510 + keep, **FEW_LONG)
    _check(w, wl.generate(w), layout="NHD")


@pytest.mark.parametrize("word", [0, 3])
def test_kept_channels_in_one_mask_word(word):
    w = wl.small(name=f"shortword{word}", batch=1, n_q_heads=8, n_kv_heads=1, keep=30, seqlens=(700,), seed=520)
    t = wl.generate(w)
    k = wl.bf16_bits_to_f32(t.k)
    k[..., 32 * word:32 * word + 32] *= 64.0
    t.k = wl.f32_to_bf16_bits(k.astype(np.float32))
    q = wl.bf16_bits_to_f32(t.q)
    t.q = wl.f32_to_bf16_bits((q / 64.0).astype(np.float32))
    _check(w, t)


@pytest.mark.parametrize("n_splits", [1, 3, 40])
def test_split_counts(n_splits):
    w = wl.small(name=f"shortsplit{n_splits}", batch=2, n_q_heads=16, n_kv_heads=2, keep=33, seqlens=(4000, 90), seed=530)
    _check(w, wl.generate(w), n_splits=n_splits)


# (eight KV heads: 32 places, of four tiles a pass; up to 160 tiles in all, or more than 64 a sequence)
@pytest.mark.parametrize("seqlens,form", [((2500,) * 4, 2), ((2600,) * 4, 1), ((700, 3000, 5, 1300, 2400, 0), 2), ((9000, 7000), 2), ((16384,), 2), ((16385,), 1)])
def test_chunks_of_more_than_one_pass(seqlens, form):
    w = wl.small(name=f"shortpass{len(seqlens)}", batch=len(seqlens), n_q_heads=64, n_kv_heads=8, keep=33, seqlens=seqlens, seed=540)
    _check(w, wl.generate(w), form=form)


@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_appended_rows(G):
    lens = (0, 1, 15, 16, 17, 255, 256, 257, 300)
    w = wl.small(name=f"shorttail{G}", batch=len(lens), n_q_heads=4 * G, n_kv_heads=4, keep=90, seqlens=(5, 0, 300, 64, 17, 0, 900, 33, 1), seed=550 + G)
    desc = make_desc(w)
    desc.tail_capacity = 300
    assert spark.call_form(desc, spark.CALL_DECODE_TAIL) == 2
    _tail_case(w, cap=300, tail_len=lens, seed=551 + G)


@pytest.mark.parametrize("G", [1, 4, 8])
def test_query_that_is_only_2_byte_aligned(G):
    w = wl.small(name=f"shortalign{G}", batch=2, n_q_heads=2 * G, n_kv_heads=2, keep=90, seqlens=(130, 0), seed=570 + G)
    t = wl.generate(w)
    rng = np.random.default_rng(G)
    cap = 40
    tk, tv = (to_dev(wl.f32_to_bf16_bits(rng.standard_normal((2, cap, 2, 128)).astype(np.float32))) for _ in range(2))
    tl = torch.tensor([40, 17], dtype=torch.int32, device="cuda")
    desc = make_desc(w)
    desc.tail_capacity = cap
    assert spark.call_form(desc, spark.CALL_DECODE_TAIL) == 2
    cu = torch.from_numpy(np.asarray(t.cu, np.int32)).cuda()
    packed = torch.empty(spark.packed_bytes(desc), dtype=torch.uint8, device="cuda")
    spark.prune(desc, to_dev(t.k), to_dev(t.qwin), cu, packed)
    outs = []
    for shift in (0, 1):
        buf = torch.zeros(t.q.size + 8, dtype=torch.int16, device="cuda")
        q = buf[shift:shift + t.q.size]
        q.copy_(to_dev(t.q).reshape(-1))
        outs.append(torch.empty((2, 2 * G, 128), dtype=torch.float32, device="cuda"))
        spark.decode_attn_tail(desc, q, packed, to_dev(t.v), cu, tk, tv, tl, outs[-1], spark.new_decode_workspace(desc))
    assert torch.isfinite(outs[0]).all() and torch.equal(outs[0], outs[1])


def test_only_appended_rows_and_none_at_all():
    w = wl.small(name="shorttail0", batch=3, n_q_heads=16, n_kv_heads=2, keep=33, seqlens=(0, 40, 0), seed=560)
    desc = make_desc(w)
    desc.tail_capacity = 20
    assert spark.call_form(desc, spark.CALL_DECODE_TAIL) == 2
    _tail_case(w, cap=20, tail_len=(20, 0, 0), seed=561)
