"""Appended rows on the matrix cores: row counts around the sixteen rows of an operand, the 64 of a wavefront and the 256 of
a block (16 and 64 where a block takes a tile), all query-group sizes, a query that is only 2-byte aligned, and scores whose query and softmax scale are far from
one (a power of two moved from one to the other changes nothing)."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
import paper_2508_15212_amd as spark
from tests.gpu_util import make_desc, to_dev
from tests.test_gpu_tail import _tail_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("keep", [26, 64])
@pytest.mark.parametrize("G", [1, 2, 4, 8, 16])
def test_row_counts(G, keep):
    lens = (1, 15, 16, 17, 32, 33, 63, 64, 65, 128, 255, 256, 257, 300)
    w = wl.small(name=f"tailrows{G}", batch=len(lens), n_q_heads=2 * G, n_kv_heads=2, keep=keep, seqlens=(0, 5) * 7, seed=440 + G)
    n_splits = 1 if keep == 26 else 0
    _tail_case(w, cap=300, tail_len=lens, seed=441 + G, n_splits=n_splits, tiles=0 if n_splits else 1 if G <= 8 else 4)


@pytest.mark.parametrize("shift", [-60, 60])
@pytest.mark.parametrize("G", [1, 4, 16])
def test_alignment_and_range(G, shift):
    w = wl.small(name=f"tailrange{G}", batch=2, n_q_heads=G, n_kv_heads=1, keep=26, seqlens=(0, 100), seed=450 + G)
    t = wl.generate(w)
    cap = 90
    rng = np.random.default_rng(G)
    tk, tv = (to_dev(wl.f32_to_bf16_bits(rng.standard_normal((2, cap, 1, 128)).astype(np.float32))) for _ in range(2))
    tl = torch.tensor([90, 37], dtype=torch.int32, device="cuda")
    cu = torch.from_numpy(np.asarray(t.cu, np.int32)).cuda()
    q = wl.bf16_bits_to_f32(t.q)

    def run(scale_by, offset):
        desc = make_desc(w)
        desc.tail_capacity, desc.softmax_scale = cap, float(np.ldexp(1.0 / np.sqrt(128.0), -scale_by))
        packed = torch.empty(spark.packed_bytes(desc), dtype=torch.uint8, device="cuda")
        spark.prune(desc, to_dev(t.k), to_dev(t.qwin), cu, packed)
        buf = torch.zeros(2 * G * 128 + 8, dtype=torch.int16, device="cuda")
        dq = buf[offset:offset + 2 * G * 128]
        dq.copy_(to_dev(wl.f32_to_bf16_bits(np.ldexp(q, scale_by).astype(np.float32))).reshape(-1))
        out = torch.empty((2, G, 128), dtype=torch.float32, device="cuda")
        spark.decode_attn_tail(desc, dq, packed, to_dev(t.v), cu, tk, tv, tl, out, spark.new_decode_workspace(desc))
        return out.cpu()

    base = run(0, 0)
    assert torch.isfinite(base).all()
    assert torch.equal(base, run(0, 1))
    assert torch.equal(base, run(shift, 0))


# (26, with a split: the appended rows' blocks of 256 rows by four wavefronts, 90: by sixteen, 64: blocks of 64 rows; G = 16 has the first only)
@pytest.mark.parametrize("keep", [26, 90, 64])
@pytest.mark.parametrize("G", [1, 2, 4, 8, 16])
def test_infinite_values(G, keep):
    """+-inf in an appended value gives +-inf in the outputs of its channel and nothing elsewhere: the probabilities go to the
    matrix cores in parts, of which some are 0.  In the row that takes the softmax of every query head, in rows in the
    middle, and in the last one."""
    lens = (90, 37, 250, 1)
    w = wl.small(name=f"tailinf{G}", batch=4, n_q_heads=G, n_kv_heads=1, keep=keep, seqlens=(0, 100, 70, 0), seed=470 + G)
    t = wl.generate(w)
    # (no score so high that an appended row's probability is 0 in float32: 0 times infinity is NaN by rights)
    t.k = wl.f32_to_bf16_bits((wl.bf16_bits_to_f32(t.k) * 0.02).astype(np.float32))
    rng = np.random.default_rng(G)
    cap = 300
    tk, tv = (rng.standard_normal((4, cap, 1, 128)).astype(np.float32) for _ in range(2))
    q = wl.bf16_bits_to_f32(t.q)
    for b in range(4):
        tk[b, 0, 0] = 0.5 * q[b].sum(0)                  # (a high score: its probability is 1, or close to it)
    finite = tv.copy()
    place = {0: 3, 20: 17, 36: 64, 89: 90, 200: 100, 249: 127}
    for row, ch in place.items():
        tv[:, row, 0, ch] = np.inf if row % 2 == 0 else -np.inf
        finite[:, row, 0, ch] = 0.0
    desc = make_desc(w, n_splits=1 if keep == 26 else 0)
    desc.tail_capacity = cap
    assert spark.call_form(desc, spark.CALL_DECODE_TAIL) == (1 if keep != 90 or G == 16 else 2)
    assert spark.call_form(desc, spark.CALL_DECODE_TAIL_TILES) == (0 if keep == 26 else 1 if keep == 64 and G <= 8 else 4)
    packed = torch.empty(spark.packed_bytes(desc), dtype=torch.uint8, device="cuda")
    cu = torch.from_numpy(np.asarray(t.cu, np.int32)).cuda()
    spark.prune(desc, to_dev(t.k), to_dev(t.qwin), cu, packed)
    out = torch.empty((4, G, 128), dtype=torch.float32, device="cuda")
    bits = lambda x: to_dev(wl.f32_to_bf16_bits(x))
    tl = np.asarray(lens, np.int32)
    spark.decode_attn_tail(desc, to_dev(t.q), packed, to_dev(t.v), cu, bits(tk), bits(tv), torch.from_numpy(tl).cuda(), out,
                           spark.new_decode_workspace(desc))
    got = out.cpu().numpy()
    _, _, a32 = oracle.window_stat(t.qwin, 1)
    ref = oracle.decode_literal_tail(t.q, oracle.prune(t.k, t.layout, a32, t.cu, keep), t.v, t.layout, t.cu,
                                     wl.f32_to_bf16_bits(tk), wl.f32_to_bf16_bits(finite), tl)
    for row, ch in place.items():
        for b in range(4):
            if row < lens[b]:
                assert np.all(got[b, :, ch] == (np.inf if row % 2 == 0 else -np.inf)), (b, row, ch)
                got[b, :, ch] = ref[b, :, ch]
    assert np.abs(got - ref).max() <= 1e-2
