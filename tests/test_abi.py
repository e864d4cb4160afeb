"""CPU-side checks of the boundary: the library loads, exports every symbol the header
declares, answers the size queries, and rejects bad descriptions without touching a GPU."""
import ctypes
import os
import re

import paper_2508_15212_amd as spark
from paper_2508_15212_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    names = set()
    for header in ("spark.h", "spark_bench.h"):
        text = open(os.path.join(ROOT, "include", header)).read()
        text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
        names |= set(re.findall(r"\b(spark_[a-z_0-9]+)\s*\(", text))
    return sorted(names)


def test_the_method_header_holds_no_measurement_aid():
    text = open(os.path.join(ROOT, "include", "spark.h")).read()
    assert "spark_probe_read" not in text


def test_library_exports_every_declared_symbol():
    lib = spark.load()
    names = _declared()
    assert set(names) == set(binding.EXPORTS)
    for n in names:
        assert getattr(lib, n) is not None


def _desc(**kw):
    d = spark.SparkDesc(batch=8, n_q_heads=32, n_kv_heads=8, head_dim=128, keep=26, window=32,
                        total_tokens=8 * 32768, k_token_stride=128, k_head_stride=128 * 8 * 32768,
                        v_token_stride=128, v_head_stride=128 * 8 * 32768)
    for k, v in kw.items():
        setattr(d, k, v)
    return d


def test_size_queries_follow_the_layout():
    d = _desc()
    rows = 8 * 32768 * 8
    # 72-byte rows at T = 26 (13 value words + 4 mask words + mu), plus header and a / 1/a
    assert spark.packed_bytes(d) == 256 + 2 * 8 * 8 * 128 * 4 + rows * 72
    assert spark.packed_bytes(_desc(keep=64)) == 256 + 2 * 8 * 8 * 128 * 4 + rows * 152
    assert spark.packed_bytes(_desc(pack_dtype=spark.PACK_INT8)) == 256 + 2 * 8 * 8 * 128 * 4 + rows * 56
    ns = spark.decode_splits(d)
    assert ns >= 1
    assert ns == 8                          # 4096 tiles x 8 heads / 512 blocks = chunks of 64 tiles; 512 / 64
    # slots: one per (chunk, q head) for at most (4096 + 2 * 8) // 64 + 8 + 1 = 73 chunks, plus one spare per
    # (batch, q head) for appended rows; 130 floats per slot; then the 8 * 8 arrival counters
    # (the counters come first, padded to 256 bytes, so their place depends on batch and KV heads only)
    assert spark.decode_workspace_bytes(d) == (73 * 32 + 8 * 32 * 1) * 130 * 4 + 256
    assert spark.decode_workspace_bytes(_desc(batch=64, total_tokens=64 * 2048)) % 256 == 0
    assert spark.decode_splits(_desc(n_splits=7)) == 7
    # partial last tile is padded to 64 tokens
    assert spark.packed_bytes(_desc(batch=1, total_tokens=65)) == 256 + 2 * 8 * 128 * 4 + 2 * 64 * 8 * 72


def test_balanced_cut_sizes_its_partial_slots_on_the_host():
    """n_splits = -1 asks for the balanced cut: 4 * (512 / KV heads) wavefronts per KV head, chunk ids
    wavefronts + 2 * batch - 1 (the size holds one more).  Batches of 32 to 256 sequences with 256 or more (batch, KV head) pairs and two
    tiles or more per wavefront get it unasked; more than 256 sequences, or 16 query heads per KV head, never do."""
    slot = 130 * 4
    small = _desc(batch=4, total_tokens=4 * 1000)
    forced = _desc(batch=4, total_tokens=4 * 1000, n_splits=-1)
    assert spark.decode_workspace_bytes(forced) == ((256 + 2 * 4) * 32 + 4 * 32) * slot + 256
    assert spark.decode_workspace_bytes(forced) > spark.decode_workspace_bytes(small)
    assert spark.decode_splits(forced) == 0 and spark.decode_splits(small) >= 1     # (0: the balanced cut)
    ragged = _desc(batch=64, total_tokens=64 * 1300)
    assert spark.decode_workspace_bytes(ragged) == ((256 + 2 * 64) * 32 + 64 * 32) * slot + 64 * 8 * 4
    assert spark.decode_workspace_bytes(_desc(batch=64, total_tokens=64 * 1300, n_splits=-1)) == \
        spark.decode_workspace_bytes(ragged)
    # a fixed split count switches it off; so do 16 query heads per KV head and more than 256 sequences
    assert spark.decode_workspace_bytes(_desc(batch=64, total_tokens=64 * 1300, n_splits=1)) == \
        (64 * 32 + 64 * 32) * slot + 64 * 8 * 4
    wide = dict(n_q_heads=128, n_kv_heads=8, batch=4, total_tokens=4 * 1000)
    assert spark.decode_workspace_bytes(_desc(n_splits=-1, **wide)) == spark.decode_workspace_bytes(_desc(**wide))
    many = dict(batch=300, total_tokens=300 * 100)
    assert spark.decode_workspace_bytes(_desc(n_splits=-1, **many)) == spark.decode_workspace_bytes(_desc(**many))
    # the caller's hint: a longest sequence within 9/8 of the average keeps one block per sequence
    # (chunks of 2 * ceil(1300 tiles * 8 heads / 512) = 42 tiles: at most (1300 + 128) // 42 + 64 + 1 = 99 of them)
    by_length = (99 * 32 + 64 * 32) * slot + 64 * 8 * 4
    assert spark.decode_workspace_bytes(_desc(batch=64, total_tokens=64 * 1300, max_seqlen=1400)) == by_length
    assert spark.decode_workspace_bytes(_desc(batch=64, total_tokens=64 * 1300, max_seqlen=1463)) > by_length
    assert spark.decode_workspace_bytes(_desc(batch=64, total_tokens=64 * 1300, max_seqlen=1400, n_splits=-1)) > by_length
    # ... and a batch with less than two tiles per wavefront (here 400 tiles for 256 wavefronts) is left alone
    assert spark.decode_splits(_desc(batch=64, total_tokens=64 * 400)) >= 1
    assert spark.decode_splits(_desc(batch=64, total_tokens=64 * 400, n_splits=-1)) == 0
    assert spark.decode_workspace_bytes(_desc(max_seqlen=-1)) == 0
    assert spark.decode_workspace_bytes(_desc(n_splits=-2)) == 0
    assert spark.decode_workspace_bytes(_desc(n_splits=4097)) == 0


def test_bad_descriptions_are_rejected_on_the_host():
    lib = spark.load()
    assert spark.packed_bytes(_desc(head_dim=64)) == 0
    assert spark.packed_bytes(_desc(keep=0)) == 0
    assert spark.packed_bytes(_desc(keep=129)) == 0
    assert spark.packed_bytes(_desc(n_q_heads=24, n_kv_heads=8)) == 0      # group of 3
    assert spark.packed_bytes(_desc(n_q_heads=30)) == 0
    # NULL pointers are caught before any launch (status 1 = invalid argument)
    d = _desc()
    assert lib.spark_prune(ctypes.byref(d), None, None, None, None, None, 0, None) == 1
    assert lib.spark_decode_attn(ctypes.byref(d), None, None, None, None, None, None, 0, None) == 1
    assert lib.spark_unpack(ctypes.byref(d), None, None, None, None, None, None, None) == 1
    assert lib.spark_prune(ctypes.byref(_desc(head_dim=64)), None, None, None, None, None, 0, None) == 2
    assert lib.spark_status_string(3) == b"workspace too small"


def test_alignment_strides_and_workspace_are_checked_before_any_launch():
    """Fake (never dereferenced) device addresses: every one of these calls must fail on the host."""
    lib = spark.load()
    d = _desc()
    A = 0x7F0000000000            # 256-byte aligned fake address
    ok_ws = spark.decode_workspace_bytes(d)
    # misaligned packed buffer / V pointer / workspace
    assert lib.spark_prune(ctypes.byref(d), A, A, A, A + 64, None, 0, None) == 1
    assert lib.spark_decode_attn(ctypes.byref(d), A, A + 8, A, A, A, A, ok_ws, None) == 1
    assert lib.spark_decode_attn(ctypes.byref(d), A, A, A + 2, A, A, A, ok_ws, None) == 1
    assert lib.spark_decode_attn(ctypes.byref(d), A, A, A, A, A, A + 4, ok_ws, None) == 1
    # workspace one byte short
    assert lib.spark_decode_attn(ctypes.byref(d), A, A, A, A, A, A, ok_ws - 1, None) == 3
    assert lib.spark_decode_workspace_init(ctypes.byref(d), A, ok_ws - 1, None) == 3
    # strides that would break 16-byte row alignment, or rows that overlap
    assert lib.spark_prune(ctypes.byref(_desc(k_token_stride=130)), A, A, A, A, None, 0, None) == 1
    assert lib.spark_prune(ctypes.byref(_desc(k_token_stride=64)), A, A, A, A, None, 0, None) == 1
    assert lib.spark_decode_attn(ctypes.byref(_desc(v_head_stride=100)), A, A, A, A, A, A, ok_ws, None) == 1
    assert lib.spark_prune(ctypes.byref(_desc(window=0)), A, A, A, A, None, 0, None) == 1
    assert lib.spark_probe_read(None, 1024, A, 4, None) == 1
    assert lib.spark_probe_read(A, 8, A, 4, None) == 1
    # K and V base pointers must be 16-byte aligned (the kernels issue 4- and 16-byte row loads)
    assert lib.spark_prune(ctypes.byref(d), A + 2, A, A, A, None, 0, None) == 1
    assert lib.spark_prune(ctypes.byref(d), A + 8, A, A, A, None, 0, None) == 1
    assert lib.spark_prune_values(ctypes.byref(_desc(keep_v=64)), A + 4, A, None) == 1
    # the cache checker rejects bad arguments before it copies anything
    assert lib.spark_check_packed(ctypes.byref(d), None, 0, None) == 1
    assert lib.spark_check_packed(ctypes.byref(d), A + 64, 0, None) == 1
    assert lib.spark_check_packed(ctypes.byref(d), A, 1, None) == 1          # keep_v = 0: there is no value cache
    assert lib.spark_check_packed(ctypes.byref(_desc(head_dim=64)), A, 0, None) == 2
    assert lib.spark_status_string(5) == b"packed cache does not match the description"


def test_value_cache_and_tail_entry_points_check_their_arguments_on_the_host():
    lib = spark.load()
    A = 0x7F0000000000
    rows = 8 * 32768 * 8
    # value cache: rows of 16 mask bytes + 2 bytes per kept entry, no statistic, no a section
    assert spark.packed_values_bytes(_desc(keep_v=64)) == 256 + rows * 144
    assert spark.packed_values_bytes(_desc(keep_v=26)) == 256 + rows * 72       # 68 -> rows are 8-byte multiples
    assert spark.packed_values_bytes(_desc()) == 0                               # keep_v = 0: values stay dense
    assert spark.packed_values_bytes(_desc(keep_v=129)) == 0
    d = _desc(keep_v=64)
    ok_ws = spark.decode_workspace_bytes(d)
    assert lib.spark_prune_values(ctypes.byref(_desc()), A, A, None) == 1        # keep_v missing
    assert lib.spark_prune_values(ctypes.byref(d), None, A, None) == 1
    assert lib.spark_prune_values(ctypes.byref(d), A, A + 64, None) == 1         # packed buffer misaligned
    assert lib.spark_prune_values(ctypes.byref(_desc(keep_v=64, v_token_stride=1 << 25)), A, A, None) == 2
    assert lib.spark_decode_attn_values(ctypes.byref(d), A, A, None, A, A, A, ok_ws, None) == 1
    assert lib.spark_decode_attn_values(ctypes.byref(_desc()), A, A, A, A, A, A, ok_ws, None) == 1
    assert lib.spark_unpack_values(ctypes.byref(d), None, None, None, None) == 1
    # appended rows: capacity enters the workspace size (one spare slot per 256 rows)
    dt = _desc(tail_capacity=600)
    assert spark.decode_workspace_bytes(dt) == (73 * 32 + 8 * 32 * 3) * 130 * 4 + 256
    ws_t = spark.decode_workspace_bytes(dt)
    assert lib.spark_decode_attn_tail(ctypes.byref(dt), A, A, A, A, None, A, A, A, A, ws_t, None) == 1
    assert lib.spark_decode_attn_tail(ctypes.byref(dt), A, A, A, A, A, None, A, A, A, ws_t, None) == 1
    assert lib.spark_decode_attn_tail(ctypes.byref(dt), A, A, A, A, A + 8, A, A, A, A, ws_t, None) == 1
    assert lib.spark_decode_attn_tail(ctypes.byref(_desc()), A, A, A, A, A, A, A, A, A, ws_t, None) == 1   # capacity 0
    assert lib.spark_decode_attn_tail(ctypes.byref(dt), A, A, A, A, A, A, A, A, A, ws_t - 1, None) == 3
    assert spark.packed_bytes(_desc(tail_capacity=-1)) == 0


def test_size_limits_of_the_description():
    assert spark.packed_bytes(_desc(batch=1, total_tokens=(1 << 31) - 256)) > 0
    assert spark.packed_bytes(_desc(batch=1, total_tokens=(1 << 31) - 255)) == 0
    assert spark.packed_bytes(_desc(batch=(1 << 18) + 1)) == 0


def test_statistics_rows_and_sampled_decode_arguments():
    lib = spark.load()
    A = 0x7F0000000000
    rows = 8 * 32768 * 8
    ds = _desc(stats=1)
    assert spark.packed_bytes(ds) == 256 + 2 * 8 * 8 * 128 * 4 + rows * 80      # 72 + mean + standard deviation
    # int8 storage: mask 16 + mu 4 + scale 4 + mean and standard deviation 8 + 7 code words 28 = 60 -> 64-byte rows
    assert spark.packed_bytes(_desc(stats=1, pack_dtype=spark.PACK_INT8)) == 256 + 2 * 8 * 8 * 128 * 4 + rows * 64
    assert spark.packed_bytes(_desc(stats=2)) == 0
    ws = spark.decode_workspace_bytes(ds)
    u64 = ctypes.c_uint64(1)
    assert lib.spark_decode_attn_sampled(ctypes.byref(_desc()), A, A, A, A, A, A, ws, 1, u64, None) == 1   # no stats
    assert lib.spark_decode_attn_sampled(ctypes.byref(ds), A, A, A, A, A, A, ws, 0, u64, None) == 1        # bad kind
    assert lib.spark_decode_attn_sampled(ctypes.byref(ds), A, A, A, A, A, A, ws, 3, u64, None) == 1
    assert lib.spark_decode_attn_sampled(ctypes.byref(ds), A, A, None, A, A, A, ws, 1, u64, None) == 1
    assert lib.spark_decode_attn_sampled(ctypes.byref(ds), A, A, A, A, A, A, ws - 1, 1, u64, None) == 3
    assert lib.spark_unpack_stats(ctypes.byref(_desc()), A, A, A, None) == 1
    assert lib.spark_unpack_stats(ctypes.byref(ds), None, A, A, None) == 1


def test_bench_traffic_table_names_profile_files_that_hold_the_figures():
    # every stored HBM-traffic figure of bench.py comes out of the profile summary the table names
    import bench
    assert bench.TRAFFIC_PROFILES
    for (workload, pack), rel in bench.TRAFFIC_PROFILES.items():
        assert os.path.exists(os.path.join(ROOT, rel)), rel
        nbytes, src = bench.measured_traffic(workload, pack)
        assert src == rel and nbytes is not None and nbytes > 0, (workload, pack)
    assert bench.measured_traffic("no_such_workload", "bf16") == (None, None)


def test_timeline_aid_checks_its_buffer_on_the_host():
    lib = spark.load()
    assert lib.spark_decode_timeline(None, 0) == 0                       # off
    assert lib.spark_decode_timeline(0x7F0000000004, 4096) == 1          # misaligned
    assert lib.spark_decode_timeline(0x7F0000000000, 32) == 1            # no room for one block
    assert lib.spark_decode_timeline(None, 0) == 0


def test_one_launch_of_the_top_p_prune_only_where_words_and_sums_can_be_told_apart():
    """The one launch files a tile's own words as 2^32 - 8192 and up: a stream must not have room for that many words."""
    form = lambda **kw: spark.call_form(_desc(**kw), spark.CALL_PRUNE_TOPP)
    fits = ((1 << 32) - 8192) // 4096 - 1                  # tiles of 64 rows of 64 words
    assert form(n_kv_heads=4, batch=1, total_tokens=64 * fits) == 1
    assert form(n_kv_heads=4, batch=1, total_tokens=64 * fits + 1) == 3
    assert form(n_kv_heads=8, batch=1, total_tokens=(1 << 31) - 256) == 3
    # few tiles, or many of four heads or more
    assert form(n_q_heads=1, n_kv_heads=1, batch=1, total_tokens=112 * 64) == 1
    assert form(n_q_heads=1, n_kv_heads=1, batch=1, total_tokens=112 * 64 + 1) == 3
    assert form(batch=1, total_tokens=2048) == 1 and form(batch=1, total_tokens=2049) == 3
    assert form(batch=1, total_tokens=256 * 64) == 1 and form(batch=1, total_tokens=255 * 64) == 3
    assert form(n_q_heads=2, n_kv_heads=2, batch=1, total_tokens=1 << 20) == 3
    assert form(total_tokens=0) == 0 and form(head_dim=64) == 0
    assert spark.call_form(_desc(), -1) == 0


def test_reported_splits_follow_the_limits_on_the_chunks():
    """A few sequences are cut into no more chunks than the chip holds blocks, a short call into no more than it has
    compute units."""
    six = dict(batch=6, total_tokens=6 * 1300, keep=32, n_q_heads=64)      # 21 tiles each, eight KV heads
    assert spark.call_form(_desc(**six), spark.CALL_DECODE) == 2
    assert spark.decode_splits(_desc(**six)) == 5                  # 32 places: 5 tiles a chunk (4 would be 36 chunks)
    assert spark.call_form(_desc(**six, n_splits=9), spark.CALL_DECODE) == 1
    assert spark.decode_splits(_desc(**six, n_splits=9)) == 9
    ten = dict(batch=10, total_tokens=10 * 8000)                   # 125 tiles each; 64 places
    assert spark.call_form(_desc(**ten), spark.CALL_DECODE) == 1
    assert spark.decode_splits(_desc(**ten)) == 6                  # (20 tiles a chunk would be 70)
    # no limit: 256 pairs and more
    assert spark.decode_splits(_desc(batch=40, total_tokens=40 * 1000, max_seqlen=1000)) == 1
    # appended rows take places of their own
    tail = dict(batch=4, total_tokens=4 * 2400, keep=33, n_q_heads=64, tail_capacity=256)
    assert spark.call_form(_desc(**tail), spark.CALL_DECODE) == 2 and spark.call_form(_desc(**tail), spark.CALL_DECODE_TAIL) == 2
    tail["tail_capacity"] = 2048
    assert spark.call_form(_desc(**tail), spark.CALL_DECODE) == 2 and spark.call_form(_desc(**tail), spark.CALL_DECODE_TAIL) == 1
    assert spark.call_form(_desc(batch=64, total_tokens=64 * 1300), spark.CALL_DECODE) == 3


def test_blocks_of_sixteen_wavefronts_only_where_they_were_measured_faster():
    form = lambda G, keep, lens, hkv=8: spark.call_form(_desc(n_q_heads=G * hkv, n_kv_heads=hkv, keep=keep, batch=len(lens), total_tokens=sum(lens)),
                                                        spark.CALL_DECODE)
    # a second pass for little, few tiles a sequence
    for G in (1, 2, 4):
        for keep in (30, 48):
            assert form(G, keep, (2000, 2200, 2400, 2600, 2800, 3000)) == 1
            assert form(G, keep, (6000, 10000)) == 1
    assert form(8, 30, (2000, 2200, 2400, 2600, 2800, 3000)) == 1 and form(8, 26, (2000, 2200, 2400, 2600, 2800, 3000)) == 1
    assert form(2, 48, (300,) * 8) == 1 and form(8, 64, (300,) * 8) == 1 and form(4, 30, (300,) * 8) == 1
    # many tiles a sequence; long rows; eight query heads
    for G in (1, 2, 4):
        assert form(G, 30, (8192,)) == 2 and form(G, 30, (65536,), 2) == 2 and form(G, 90, (1024,)) == 2 and form(G, 90, (16384,)) == 1
        assert form(G, 26, (8192,)) == 1
    assert form(8, 30, (100,)) == 2 and form(8, 26, (8192,)) == 2 and form(8, 64, (16384,)) == 1 and form(8, 26, (16384,)) == 2


def _tiles(lens, tail=False, G=4, hkv=8, **kw):
    """Tiles of a block of the decode call: 1 is a block per tile."""
    d = _desc(n_q_heads=G * hkv, n_kv_heads=hkv, batch=len(lens), total_tokens=sum(lens), **kw)
    return spark.call_form(d, spark.CALL_DECODE_TAIL_TILES if tail else spark.CALL_DECODE_TILES)


def test_the_block_per_tile_can_be_told_from_blocks_of_four():
    assert _tiles((1024,), keep=64) == 1 and _tiles((1024,), keep=64, tail=True, tail_capacity=64) == 1
    assert _tiles((1024,), keep=64, tail=True, tail_capacity=1 << 14) == 4      # (256 blocks of appended rows a KV head)
    assert _tiles((1024,), keep=64, G=16) == 4
    # (eight query heads with short rows never: also where there are fewer tiles than sequences)
    assert _tiles((3,) * 11 + (1, 1, 0), keep=26, G=8) == 4 and _tiles((1024,), keep=26, G=8) == 4
    assert _tiles((32768,) * 8) == 64 and _tiles((1024,), keep=64, n_splits=2) == 0 and _tiles((1300,) * 64) == 0


def test_room_for_appended_rows_is_what_calls_with_appended_rows_use():
    """Four sequences of 400 tokens take a block per tile without appended rows, and blocks of four with many: their workspace
    has slots for 256 appended rows each, as those blocks take them, not for 64."""
    slot = 130 * 4
    for capacity in (4096, 32768):
        kw = dict(batch=4, total_tokens=4 * 400, keep=64, tail_capacity=capacity)
        assert spark.call_form(_desc(**kw), spark.CALL_DECODE_TILES) == 1 and spark.call_form(_desc(**kw), spark.CALL_DECODE_TAIL_TILES) == 4
        # (chunks: at most (25 tiles + 2 * 4) // 4 + 4 + 1)
        assert spark.decode_workspace_bytes(_desc(**kw)) == (13 * 32 + 4 * 32 * (capacity // 256)) * slot + 256
    # with few: slots for 64 rows each, and as many chunks as tiles that four sequences can span, and one
    kw = dict(batch=4, total_tokens=4 * 400, keep=64, tail_capacity=128)
    assert spark.call_form(_desc(**kw), spark.CALL_DECODE_TAIL_TILES) == 1
    assert spark.decode_workspace_bytes(_desc(**kw)) == ((25 + 4) * 32 + 4 * 32 * 2) * slot + 256


def test_a_block_per_tile_only_where_it_was_measured_faster():
    """Both sides of every limit: tiles that one sequence can have, blocks, tokens a sequence, row lengths."""
    n = lambda tiles: (64 * tiles,)
    for G, keep, most, hkv in ((1, 64, 96, 2), (2, 64, 64, 4), (4, 64, 32, 8), (8, 64, 24, 8), (2, 38, 48, 4), (4, 38, 20, 8), (8, 38, 20, 8), (2, 26, 32, 4), (4, 26, 20, 8), (4, 25, 20, 8), (1, 26, 32, 4), (1, 38, 32, 4), (1, 33, 96, 4), (2, 33, 64, 8), (4, 33, 36, 8),
                               (1, 20, 96, 4), (4, 28, 36, 8)):
        assert _tiles(n(most), keep=keep, G=G, hkv=hkv) == 1 and _tiles(n(most + 1), keep=keep, G=G, hkv=hkv) > 1, (G, keep)
        # without a longest length one sequence of several has four fifths of the tiles; with one, it has those and one more at a seam
        several = lambda tiles: (64 * tiles - 2 * 240, 240, 240)
        assert _tiles(several(most * 5 // 4), keep=keep, G=G, hkv=2) == 1 and _tiles(several(most * 5 // 4 + 1), keep=keep, G=G, hkv=2) == 4, (G, keep)
        for max_seqlen, tiles in ((64 * (most - 1), 1), (64 * (most - 1) + 1, 4)):
            assert _tiles(several(most * 5 // 4 + 1), keep=keep, G=G, hkv=2, max_seqlen=max_seqlen) == tiles, (G, keep, max_seqlen)
        # appended rows are merged too: 64 a block
        assert _tiles(n(most - 3), True, keep=keep, G=G, hkv=2, tail_capacity=192) == 1 and _tiles(n(most - 2), True, keep=keep, G=G, hkv=2, tail_capacity=192) == 4
    # blocks of the cache: 512, 256 with eight query heads, 704 for one and two with rows of any length
    assert _tiles((64 * 63,), keep=64, G=1) == 1 and _tiles((64 * 64,), keep=64, G=1) == 4
    for hkv, G, n in ((16, 4, 30), (8, 8, 30)):
        assert _tiles((64 * n - 900, 900), keep=64, G=G, max_seqlen=1020, hkv=hkv) == 1 and _tiles((64 * n - 836, 900), keep=64, G=G, max_seqlen=1020, hkv=hkv) == 4
    assert _tiles((64 * 50, 64 * 36), keep=33, G=1, hkv=8) == 1 and _tiles((64 * 50, 64 * 37), keep=33, G=1, hkv=8) == 4
    assert _tiles((64 * 30, 64 * 32), keep=33, G=4, hkv=8, max_seqlen=2048) == 1 and _tiles((64 * 30, 64 * 33), keep=33, G=4, hkv=8, max_seqlen=2048) == 4
    # short sequences are one block of four tiles, with appended rows two
    for keep, G, tokens in ((64, 1, 240), (64, 2, 200), (64, 4, 200), (64, 8, 200), (33, 4, 200), (39, 1, 200), (26, 2, 240), (38, 4, 240)):
        assert _tiles((tokens - 1,), keep=keep, G=G) == 4 and _tiles((tokens,), keep=keep, G=G) == 1, (keep, G)
        assert _tiles((0, 2 * tokens - 1), keep=keep, G=G) == 4 and _tiles((0, 2 * tokens), keep=keep, G=G) == 1, (keep, G)
        assert _tiles((tokens - 1,), True, keep=keep, G=G, tail_capacity=64) == 1, (keep, G)
    assert _tiles((1,), keep=40, G=1) == 1 and _tiles((190,) * 9, keep=40, G=1) == 4 and _tiles((240,) * 9, keep=40, G=1) == 1      # (256 blocks)
    # short rows with kernels of their own and eight query heads, one with int8 codes of 26, eight with rows of any length: never
    for keep, G, pack in ((25, 8, 0), (26, 8, 0), (26, 1, spark.PACK_INT8), (33, 8, 0), (64, 16, 0)):
        assert _tiles((512,), keep=keep, G=G, pack_dtype=pack) == 4 and _tiles((512,), True, keep=keep, G=G, pack_dtype=pack, tail_capacity=64) == 4, (keep, G)
    assert _tiles((512,), keep=25, G=1, pack_dtype=spark.PACK_INT8) == 1       # (no kernel of its own)
    # one long conversation among short ones
    assert _tiles((5000, 100, 100, 100), keep=64) == 4 and _tiles((40000,) + (200,) * 21, keep=64, hkv=1) == 4
