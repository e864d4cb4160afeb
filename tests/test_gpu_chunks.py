"""Decode of a few ragged sequences whose shares, rounded up one by one, would be more blocks than the chip holds at once:
the kernel takes longer chunks.  Against the CPU oracle, with and without appended rows, with packed values, and where the
limit is met exactly or by one block."""
import numpy as np
import pytest

import oracle
import workloads as wl
from tests.gpu_util import run_gpu_case
from tests.test_gpu_tail import _tail_case

pytestmark = pytest.mark.gpu
MAX_ABS, MEAN_ABS = 1e-2, 1e-3


def _check(w):
    t = wl.generate(w)
    res = run_gpu_case(w, t, want_unpack=False, want_bf16=False)
    _, _, a32 = oracle.window_stat(t.qwin, w.n_kv_heads)
    ref = oracle.decode_literal(t.q, oracle.prune(t.k, t.layout, a32, t.cu, w.keep), t.v, t.layout, t.cu)
    err = np.abs(res["out_f32"].astype(np.float64) - ref)
    assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS


# 32 KV heads: at most sixteen chunks; the first three batches would have 21, 17 and 16 of four tiles, the fourth 20
@pytest.mark.parametrize("keep", [26, 33])
@pytest.mark.parametrize("seqlens", [(560,) * 7, (0, 900, 5, 1300, 700, 0, 730), (1024, 1024, 1024, 1024), (500, 0, 512, 499, 530, 1, 520, 540)[:7]])
def test_more_chunks_than_resident_blocks(seqlens, keep):
    w = wl.small(name=f"chunks{len(seqlens)}", batch=len(seqlens), n_q_heads=32, n_kv_heads=32, keep=keep, seqlens=seqlens, seed=420 + keep)
    _check(w)


def test_one_sequence_one_chunk_too_many():
    # three KV heads: 1024 tiles in chunks of six would be 171, and 170 fit
    _check(wl.small(name="chunk1", batch=1, n_q_heads=3, n_kv_heads=3, keep=26, seqlens=(65536,), seed=431))


def test_with_appended_rows():
    w = wl.small(name="chunktail", batch=7, n_q_heads=32, n_kv_heads=32, keep=26, seqlens=(560, 40, 700, 0, 610, 570, 580), seed=432)
    _tail_case(w, cap=300, tail_len=(300, 0, 17, 256, 257, 1, 0), seed=433)
