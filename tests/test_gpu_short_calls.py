"""Decode of short calls by blocks of sixteen wavefronts, sixteen tokens a wavefront, four lanes a row: row lengths whose words
end in every place of a section, rows whose kept channels all lie in one mask word, sequence ends inside the sixteen tokens,
empty sequences, chunks of more than one pass, appended rows around the sixteen of a wavefront and the 256 of a block, and the
merge of one partial and of many.  Against the CPU oracle; tolerance as for plain decode."""
import numpy as np
import pytest

import oracle
import workloads as wl
import paper_2508_15212_amd as spark
from tests.gpu_util import run_gpu_case
from tests.test_gpu_tail import _tail_case

pytestmark = pytest.mark.gpu
MAX_ABS, MEAN_ABS = 1e-2, 1e-3


def _check(w, t, pack=spark.PACK_BF16, n_splits=0, layout="HND"):
    res = run_gpu_case(w, t, layout=layout, pack=pack, n_splits=n_splits, want_unpack=False)
    _, _, a32 = oracle.window_stat(t.qwin, w.n_kv_heads)
    pr = oracle.prune(t.k, t.layout, a32, t.cu, w.keep)
    pr = oracle.quant_int8(pr) if pack == spark.PACK_INT8 else pr
    ref = oracle.decode_literal(t.q, pr, t.v, t.layout, t.cu)
    err = np.abs(res["out_f32"].astype(np.float64) - ref)
    assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS, (err.max(), err.mean())
    # (half a unit of bf16's last place is 2^-9 of a value at most)
    assert np.abs(res["out_bf16"] - res["out_f32"]).max() <= 2.0 ** -8 * np.abs(res["out_f32"]).max()


# (enough KV heads that the call is not too short for its query-group size: 66 tiles each)
@pytest.mark.parametrize("pack", [spark.PACK_BF16, spark.PACK_INT8])
@pytest.mark.parametrize("G,Hkv", [(1, 8), (2, 8), (4, 8), (8, 1)])
@pytest.mark.parametrize("keep", [1, 27, 66, 67, 126, 128])
def test_row_lengths(keep, G, Hkv, pack):
    w = wl.small(name=f"short{keep}_{G}", batch=6, n_q_heads=G * Hkv, n_kv_heads=Hkv, keep=keep,
                 seqlens=(1, 1700, 0, 15, 2033, 451), seed=500 + keep + G)
    _check(w, wl.generate(w), pack)


@pytest.mark.parametrize("keep", [26, 64, 38])
def test_eight_query_heads_instantiated_lengths(keep):
    w = wl.small(name=f"short8_{keep}", batch=3, n_q_heads=64, n_kv_heads=8, keep=keep, seqlens=(2000, 17, 2500), seed=510 + keep)
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


@pytest.mark.parametrize("seqlens", [(3000,) * 4, (700, 3000, 5, 1300, 2400, 0)])
def test_chunks_of_more_than_one_pass(seqlens):
    w = wl.small(name=f"shortpass{len(seqlens)}", batch=len(seqlens), n_q_heads=32, n_kv_heads=8, keep=33, seqlens=seqlens, seed=540)
    _check(w, wl.generate(w))


@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_appended_rows(G):
    lens = (0, 1, 15, 16, 17, 255, 256, 257, 300)
    w = wl.small(name=f"shorttail{G}", batch=len(lens), n_q_heads=4 * G, n_kv_heads=4, keep=70, seqlens=(5, 0, 300, 64, 17, 0, 900, 33, 1), seed=550 + G)
    _tail_case(w, cap=300, tail_len=lens, seed=551 + G)


def test_only_appended_rows_and_none_at_all():
    w = wl.small(name="shorttail0", batch=3, n_q_heads=16, n_kv_heads=2, keep=33, seqlens=(0, 40, 0), seed=560)
    _tail_case(w, cap=20, tail_len=(20, 0, 0), seed=561)
