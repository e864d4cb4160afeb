"""GPU parity for value-cache channel pruning (the appendix extension that prunes keys and values
together): kept sets and kept entries bit for bit against the CPU oracle; decode over both packed
caches within the decode tolerance (max |err| <= 1e-2, mean |err| <= 1e-3)."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
import paper_2508_15212_amd as spark
from tests.gpu_util import make_desc, to_dev

pytestmark = pytest.mark.gpu


def _prune_values_gpu(w, v_bits, Tv, layout="HND"):
    v = v_bits if layout == "HND" else np.ascontiguousarray(v_bits.transpose(1, 0, 2))
    desc = make_desc(w, layout)
    desc.keep_v = Tv
    dv = to_dev(v)
    packed_v = torch.empty(max(spark.packed_values_bytes(desc), 256), dtype=torch.uint8, device="cuda")
    spark.prune_values(desc, dv, packed_v)
    mask = torch.empty((w.total, w.n_kv_heads, 4), dtype=torch.int32, device="cuda")
    vals = torch.empty((w.total, w.n_kv_heads, Tv), dtype=torch.int16, device="cuda")
    spark.unpack_values(desc, packed_v, mask, vals)
    torch.cuda.synchronize()
    return desc, packed_v, mask.cpu().numpy().view(np.uint32), vals.cpu().numpy().view(np.uint16)


@pytest.mark.parametrize("Tv", [1, 26, 63, 64, 65, 96, 127, 128])
def test_value_selection_matches_oracle(Tv):
    w = wl.small(name=f"values{Tv}", seqlens=(130, 321), seed=200 + Tv)
    t = wl.generate(w)
    pv = oracle.prune_values(t.v, t.layout, Tv)
    print(f"{w.name}: rows={w.total * w.n_kv_heads} near-ties(<1e-6)={pv.near_ties()}")
    _, _, mask, vals = _prune_values_gpu(w, t.v, Tv)
    assert np.array_equal(mask, pv.mask)
    assert np.array_equal(vals, pv.kept)


@pytest.mark.parametrize("layout", ["HND", "NHD"])
def test_value_selection_layouts_ties_zero_rows(layout):
    w = wl.small(name=f"values_ties_{layout}", batch=2, n_q_heads=4, n_kv_heads=2, seqlens=(150, 43), seed=230)
    t = wl.generate(w)
    rng = np.random.default_rng(230)
    vq = rng.integers(-2, 3, size=t.v.shape).astype(np.float32)      # a handful of magnitudes: ties at most cuts
    vq[:, 10:20, :] = 0.0                                            # all-zero rows keep channels 0..Tv-1
    vq[:, 30:40, :] = -1.5                                           # all-equal rows
    vbits = wl.f32_to_bf16_bits(vq)
    pv = oracle.prune_values(vbits, "HND", 48)
    assert pv.near_ties() > 0.5 * pv.gap.size
    _, _, mask, vals = _prune_values_gpu(w, vbits, 48, layout)
    assert np.array_equal(mask, pv.mask)
    assert np.array_equal(vals, pv.kept)


MAX_ABS, MEAN_ABS = 1e-2, 1e-3


def _decode_kv_case(w, Tv, t=None, n_splits=0, layout="HND", int8=False):
    """prune keys, prune values, decode over both packed caches; compare with the oracle."""
    t = wl.generate(w) if t is None else t
    _, _, a32 = oracle.window_stat(t.qwin, w.n_kv_heads)
    pr = oracle.prune(t.k, t.layout, a32, t.cu, w.keep)
    if int8:
        pr = oracle.quant_int8(pr)
    pv = oracle.prune_values(t.v, t.layout, Tv)
    ref = oracle.decode_literal(t.q, pr, oracle.expand_values(pv), "NHD", t.cu)

    k = t.k if layout == "HND" else np.ascontiguousarray(t.k.transpose(1, 0, 2))
    desc, packed_v, mask_v, vals_v = _prune_values_gpu(w, t.v, Tv, layout)
    assert np.array_equal(mask_v, pv.mask) and np.array_equal(vals_v, pv.kept)
    desc.n_splits = n_splits
    if int8:
        desc.pack_dtype = spark.PACK_INT8
    dk, dqw, dq = to_dev(k), to_dev(t.qwin), to_dev(t.q)
    dcu = torch.from_numpy(np.asarray(t.cu, np.int32)).cuda()
    packed = torch.empty(max(spark.packed_bytes(desc), 256), dtype=torch.uint8, device="cuda")
    spark.prune(desc, dk, dqw, dcu, packed)
    ws = spark.new_decode_workspace(desc)
    out = torch.empty((w.batch, w.n_q_heads, w.head_dim), dtype=torch.float32, device="cuda")
    spark.decode_attn_values(desc, dq, packed, packed_v, dcu, out, ws)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    err = np.abs(got.astype(np.float64) - ref)
    print(f"{w.name} Tv={Tv}: decode max|err|={err.max():.3e} mean|err|={err.mean():.3e}")
    assert np.all(np.isfinite(got))
    assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS
    return got, ref


@pytest.mark.parametrize("T,Tv", [(26, 64), (26, 38), (26, 26), (64, 64), (64, 38), (38, 64), (26, 100), (38, 77),
                                  (26, 1), (64, 128), (128, 128)])
def test_decode_over_pruned_keys_and_values(T, Tv):
    _decode_kv_case(wl.small(name=f"kv{T}_{Tv}", keep=T, seqlens=(130, 321), seed=300 + T + Tv), Tv)


@pytest.mark.parametrize("G,Hkv", [(1, 2), (2, 2), (8, 2), (16, 1)])
def test_decode_values_group_sizes(G, Hkv):
    _decode_kv_case(wl.small(name=f"kv_gqa{G}", n_q_heads=G * Hkv, n_kv_heads=Hkv, keep=26, seqlens=(257, 64, 190),
                             batch=3, seed=340 + G), 64)


def test_decode_values_ragged_empty_single_and_layout():
    w = wl.small(name="kv_ragged", batch=6, seqlens=(0, 1, 63, 64, 65, 0), keep=26, seed=360)
    got, _ = _decode_kv_case(w, 64)
    assert np.all(got[0] == 0) and np.all(got[5] == 0)
    _decode_kv_case(wl.small(name="kv_nhd", seqlens=(333, 129), seed=361), 64, layout="NHD")


@pytest.mark.parametrize("ns", [1, 3, 7])
def test_decode_values_split_counts(ns):
    _decode_kv_case(wl.small(name=f"kv_splits{ns}", batch=2, seqlens=(1500, 700), keep=26, seed=370), 64, n_splits=ns)


def test_keep_all_values_equals_dense_value_decode():
    """Tv = D stores every entry: the result must agree with the dense-value entry point."""
    from tests.gpu_util import run_gpu_case
    w = wl.small(name="kv_all", keep=26, seqlens=(300, 141), seed=380)
    t = wl.generate(w)
    got, _ = _decode_kv_case(w, 128, t=t)
    dense = run_gpu_case(w, t, want_unpack=False, want_bf16=False)["out_f32"]
    assert np.abs(got - dense).max() < 1e-5


@pytest.mark.parametrize("T,Tv", [(26, 64), (26, 26), (26, 100), (64, 64), (38, 38), (1, 5)])
def test_int8_keys_with_pruned_values(T, Tv):
    """Kept key entries stored as int8 codes with a per-row scale, kept value entries as bf16."""
    _decode_kv_case(wl.small(name=f"kv_int8_{T}_{Tv}", keep=T, seqlens=(130, 321), seed=390 + T + Tv), Tv, int8=True)
    if T == 26 and Tv == 64:
        _decode_kv_case(wl.small(name="kv_int8_g8", n_q_heads=16, n_kv_heads=2, keep=26, seqlens=(257, 64), seed=399), 64,
                        int8=True)


@pytest.mark.parametrize("G,Hkv", [(1, 2), (4, 2), (8, 1), (16, 1)])
@pytest.mark.parametrize("Tv", [25, 71, 72, 73, 74, 95, 96, 97, 98])
def test_decode_over_value_rows_around_the_short_row_limit(Tv, G, Hkv):
    """Rows of any length are parked in LDS at one of two strides; several tiles a wavefront, a ragged tail."""
    w = wl.small(name=f"values_rows{Tv}", n_q_heads=G * Hkv, n_kv_heads=Hkv, keep=26, batch=2, seqlens=(1100, 77), seed=260 + Tv)
    _decode_kv_case(w, Tv, n_splits=1)
