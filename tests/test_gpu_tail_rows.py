"""Appended rows on the matrix cores: row counts around the sixteen rows of an operand, the 64 of a wavefront and the 256 of
a block, all query-group sizes, a query that is only 2-byte aligned, and scores whose query and softmax scale are far from
one (a power of two moved from one to the other changes nothing)."""
import numpy as np
import pytest
import torch

import workloads as wl
import paper_2508_15212_amd as spark
from tests.gpu_util import make_desc, to_dev
from tests.test_gpu_tail import _tail_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G", [1, 2, 4, 8, 16])
def test_row_counts(G):
    lens = (1, 15, 16, 17, 32, 33, 63, 64, 65, 128, 255, 256, 257, 300)
    w = wl.small(name=f"tailrows{G}", batch=len(lens), n_q_heads=2 * G, n_kv_heads=2, keep=26, seqlens=(0, 5) * 7, seed=440 + G)
    _tail_case(w, cap=300, tail_len=lens, seed=441 + G)


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
