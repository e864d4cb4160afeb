"""GPU parity of the top-p selection where its parts meet: token counts around a wavefront's four and sixteen rows and
the tile of 64, saliencies that crowd into one counting bin (finer levels, key-by-key end, ties), and keys spread
below all counting bins.  Counts, masks and kept entries are compared bit for bit (see test_gpu_topp)."""
import numpy as np
import pytest

import workloads as wl
from tests.test_gpu_topp import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens", [(1,), (3, 1), (4,), (5, 11), (16,), (17,), (31, 1, 17), (63,), (64, 1), (65,), (15, 0, 33, 130)])
def test_row_counts_around_steps_wavefronts_and_tiles(lens):
    w = wl.small(name="topprows", batch=len(lens), seqlens=lens, seed=400 + sum(lens))
    t = wl.generate(w)
    _run(w, t)
    _run(w, t, layout="NHD", decode=False)


@pytest.mark.parametrize("p_bp", [1, 40, 3000, 9900, 9999, 10000])
@pytest.mark.parametrize("steps", [0, 1, 128])
def test_saliencies_in_one_bin(steps, p_bp):
    """Channel weights 1 + n 2^-14 (n up to `steps`) on rows of equal or nearly equal magnitude: up to 128 different
    saliencies, and ties of them, within one counting bin and within the finer ones."""
    w = wl.small(name="toppbin", batch=1, n_q_heads=4, n_kv_heads=1, seqlens=(70,), seed=431)
    t = wl.generate(w)
    rng = np.random.default_rng(steps)
    q = np.ones(t.qwin.shape, np.float32)                 # [1, 4, window, 128]
    ones = rng.integers(0, steps + 1, 128) * (q.shape[1] * q.shape[2]) // 128
    flat = q.reshape(-1, 128)
    for j in range(128):
        flat[:ones[j], j] = 1.0 + 2.0 ** -7
    t.qwin = wl.f32_to_bf16_bits(q)
    k = np.ones((1, 70, 128), np.float32) * np.exp2(rng.integers(-40, 40, (1, 70, 1))).astype(np.float32)
    k[0, 1::5, ::2] *= 1.0 + 2.0 ** -7
    k[0, 2::5, :3] *= 512.0                               # ... under three large keys
    k[0, 3::5, :64] = 0.0
    k *= rng.choice([-1.0, 1.0], k.shape)
    t.k = wl.f32_to_bf16_bits(k.astype(np.float32))
    _run(w, t, p_bp)


@pytest.mark.parametrize("p_bp", [9900, 9999, 10000])
def test_keys_below_the_bins(p_bp):
    """One large key and the others up to 23 octaves below it, one wavefront step mixing such rows with ordinary and
    with subnormal ones."""
    w = wl.small(name="toppdeep", batch=2, n_q_heads=4, n_kv_heads=1, seqlens=(66, 31), seed=432)
    t = wl.generate(w)
    rng = np.random.default_rng(5)
    k = wl.bf16_bits_to_f32(t.k).copy()
    for r in range(0, 97, 2):
        k[0, r] *= np.exp2(rng.uniform(-23.5, -15.0, 128)).astype(np.float32)
        k[0, r, rng.integers(128)] = 3.0
    k[0, 5::8] = k[0, 5::8] * np.float32(1e-37) * np.float32(1e-2)
    t.k = wl.f32_to_bf16_bits(k)
    _run(w, t, p_bp, decode=False)
