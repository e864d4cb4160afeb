"""GPU parity of the fixed-count selection where the number of wavefronts per tile changes (quarters of all
tiles up to 1280 of values and 1408 of keys; halves up to 3072, quarters of the last 512; beyond, halves of 1536, whole tiles in front), partly filled last tiles and sequence ends inside a tile included."""
import pytest

import workloads as wl
from tests.test_gpu_prune_rows import _keys, _values

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [26, 120])
@pytest.mark.parametrize("hkv,tokens", [(1, 1280 * 64), (3, 427 * 64 - 7), (2, 704 * 64), (1, 1409 * 64 - 30), (4, 768 * 64), (7, 439 * 64 - 1)])
# 1280, 1281, 1408, 1409, 3072, 3073 tiles
def test_tiles_around_the_changes(hkv, tokens, T):
    w = wl.small(name=f"shares{hkv}x{tokens}", keep=T, batch=3, n_q_heads=hkv, n_kv_heads=hkv, seqlens=(tokens // 2, 0, tokens - tokens // 2),
                 seed=560 + hkv)
    t = wl.generate(w)
    _keys(w, t)
    _keys(w, t, int8=True, layout="NHD")
    _values(w, t, T)
