"""GPU parity of the fixed-count selection where its parts meet: token counts around the four rows of a step, the eight
of a group, the sixteen that are written together and the tile of 64; keep counts at the ends of their range; rows
whose T-th saliency lies outside the counting window (large jumps from row to row, zero rows, plateaus) or shares its
bin with many others.  Masks, kept entries, codes and scales bit for bit."""
import numpy as np
import pytest

import oracle
import workloads as wl
import paper_2508_15212_amd as spark
from tests.gpu_util import run_gpu_case
from tests.test_gpu_parity import _check_prune
from tests.test_gpu_values import _prune_values_gpu

pytestmark = pytest.mark.gpu


def _keys(w, t, int8=False, layout="HND"):
    _, _, a32 = oracle.window_stat(t.qwin, w.n_kv_heads)
    pr = oracle.prune(t.k, t.layout, a32, t.cu, w.keep)
    if int8:
        pr = oracle.quant_int8(pr)
    res = run_gpu_case(w, t, layout=layout, pack=spark.PACK_INT8 if int8 else spark.PACK_BF16, want_bf16=False)
    _check_prune(res, a32, pr, int8)


def _values(w, t, Tv):
    pv = oracle.prune_values(t.v, t.layout, Tv)
    _, _, mask, vals = _prune_values_gpu(w, t.v, Tv)
    assert np.array_equal(mask, pv.mask) and np.array_equal(vals, pv.kept)


@pytest.mark.parametrize("lens", [(1,), (3, 2), (4,), (7, 1, 1), (9,), (15,), (16, 1), (17, 30), (63,), (64,), (65, 0, 62), (1, 47, 81)])
def test_row_counts_around_steps_groups_and_tiles(lens):
    w = wl.small(name="rows", batch=len(lens), seqlens=lens, seed=500 + sum(lens))
    t = wl.generate(w)
    _keys(w, t)
    _keys(w, t, int8=True, layout="NHD")
    _values(w, t, 38)


@pytest.mark.parametrize("T", [1, 2, 3, 4, 5, 6, 7, 9, 63, 125, 126, 127, 128])
def test_keep_counts(T):
    w = wl.small(name=f"rowsT{T}", keep=T, batch=2, seqlens=(83, 50), seed=520 + T)
    t = wl.generate(w)
    _keys(w, t)
    _keys(w, t, int8=True)
    _values(w, t, T)


@pytest.mark.parametrize("T", [1, 26, 64, 126])
@pytest.mark.parametrize("kind", ["jumps", "plateaus", "one_bin", "zeros", "two_scales"])
def test_rows_the_counting_window_does_not_fit(kind, T):
    w = wl.small(name=f"rows_{kind}", keep=T, batch=2, n_q_heads=4, n_kv_heads=2, seqlens=(70, 141), seed=540 + T)
    t = wl.generate(w)
    rng = np.random.default_rng(T)
    for name in ("k", "v"):
        x = wl.bf16_bits_to_f32(getattr(t, name)).copy()              # [2, 211, 128]
        rows = x.shape[:2]
        if kind == "jumps":          # every row at a magnitude of its own, subnormal products among them
            x *= np.exp2(rng.integers(-100, 60, rows)).astype(np.float32)[..., None]
        elif kind == "plateaus":     # a few magnitudes far apart: ties at most cuts, the mean far from the cut
            x = np.exp2(rng.choice([-30, -3, 0, 20], x.shape)).astype(np.float32) * np.sign(x + 0.5)
        elif kind == "one_bin":      # nearly equal magnitudes (channel weights made nearly equal below)
            x = np.where(rng.random(x.shape) < 0.5, 1.0, 1.0 + 2.0 ** -7).astype(np.float32) * np.sign(x + 0.5)
        elif kind == "zeros":        # from no zero to all zero
            x[rng.random(x.shape) < rng.choice([0.0, 0.3, 0.9, 1.0], rows)[..., None]] = 0.0
        else:                        # half of the channels thirty octaves below the others
            x[..., 1::2] *= np.float32(2.0 ** -30)
        setattr(t, name, wl.f32_to_bf16_bits(x.astype(np.float32)))
    if kind == "one_bin":
        t.qwin = wl.f32_to_bf16_bits(np.where(rng.random(t.qwin.shape) < 0.5, 1.0, 1.0 + 2.0 ** -7).astype(np.float32))
    for int8 in (False, True):
        _keys(w, t, int8)
    _values(w, t, T)


@pytest.mark.parametrize("T", [4, 5, 11, 12, 99, 100, 115, 116, 125, 126])
@pytest.mark.parametrize("outliers", [0, 8])
def test_keep_counts_where_the_digit_changes(T, outliers):
    w = wl.small(name=f"rowsdigit{T}", keep=T, batch=3, seqlens=(130, 1, 95), n_outlier=outliers, seed=560 + T)
    t = wl.generate(w)
    k = wl.bf16_bits_to_f32(t.k).copy()
    k[:, 40:60] *= np.exp2(np.random.default_rng(T).integers(-60, 60, (1, 20, 1))).astype(np.float32)
    t.k = wl.f32_to_bf16_bits(k)
    _keys(w, t)
    _keys(w, t, int8=True, layout="NHD")
    _values(w, t, T)
