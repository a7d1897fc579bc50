"""The tile scheduler on the host (no GPU): vfm_schedule_units runs the launchers' unit map and
the kernels' own block -> (head, tile) -> rows mapping on the CPU.  Checked here: every (head,
token) is handed out exactly once, no tile straddles a clip (cross-clip blocks are never
enumerated), clips go longest first, the grid is padded by fewer than 8 idle workgroups, and
each XCD gets one contiguous run of units, or, where units are dealt out, its share of every clip."""
import heapq

import numpy as np
import pytest

from paper_2503_12964_amd import binding, workloads as W

XCDS = 8


def _units_in_order(units):
    """Workgroup b belongs to XCD b % 8 and is that XCD's (b // 8)-th: list the live units in
    the order XCD 0's run, XCD 1's run, ... (the head-major unit numbering of a contiguous map)."""
    chunk = len(units) // XCDS
    order = [units[x + XCDS * i] for x in range(XCDS) for i in range(chunk)]
    return [tuple(int(v) for v in u) for u in order]


def _dealing_gain(lens, heads, rows):
    """How much later the contiguous order of these clips' units ends than the dealt one: units handed in
    order to the 32 CUs of an XCD, each taking its clip's length, a quarter of that by its rows.  None: every
    CU has at most one unit, or there is nothing to even out.  Beyond two units per CU: the heaviest XCD's
    work against the mean."""
    live = sorted((int(n) for n in lens if n > 0), reverse=True)
    if heads % XCDS == 0 or len(set(live)) < 2:
        return None
    tiles = [n * (0.75 + 0.25 * min(rows, n - t) / rows) for n in live for t in range(0, n, rows)]
    chunk = -(-len(tiles) * heads // XCDS)
    if chunk <= 32:
        return None
    whole = tiles * heads
    parts = [whole[x * chunk:(x + 1) * chunk] for x in range(XCDS)]
    if chunk > 64:
        return max(map(sum, parts)) * XCDS / sum(whole)

    def end(units):
        cus = [0.0] * 32
        for u in units:
            heapq.heapreplace(cus, cus[0] + u)
        return max(cus)

    return max(map(end, parts)) / end([t for t in tiles for _ in range(heads)][::XCDS])


def _check(cu, heads, rows, units=None):
    """cu: boundaries of one launch's clips (absolute packed positions; cu[0] may be > 0 when the
    launch is one run of a longer call); units: that launch's grid."""
    cu = np.asarray(cu, dtype=np.int64)
    if units is None:
        units = binding.vfm_schedule_units(cu, heads, rows)
    base = int(cu[0])
    cu = cu - base
    units = np.array(units, dtype=np.int64)
    units[units[:, 0] >= 0, 1] -= base
    total = int(cu[-1])
    lens = np.diff(cu)
    n_tiles = int(sum((n + rows - 1) // rows for n in lens))
    assert len(units) % XCDS == 0
    assert len(units) == XCDS * ((n_tiles * heads + XCDS - 1) // XCDS)
    gain = _dealing_gain(lens, heads, rows)
    # the order is told by the second workgroup: the first tile's next head, or the second XCD's run
    dealt = gain is not None and [int(v) for v in units[1]] == [1 % heads, *(int(v) for v in units[0][1:])]
    if gain is not None and abs(gain - 1.03) > 1e-3:
        assert dealt == (gain > 1.03)
    ordered = [tuple(int(v) for v in u) for u in units] if dealt else _units_in_order(units)
    live = [u for u in ordered if u[0] >= 0]
    assert len(live) == n_tiles * heads and len(units) - len(live) < XCDS
    # idle workgroups only at the end of the numbering (the last XCD's run is the short one)
    assert ordered[:len(live)] == live
    cover = np.zeros((heads, total), dtype=np.int32)
    clip_of = np.repeat(np.arange(len(lens)), lens)
    for head, first, n in live:
        assert 0 <= head < heads and 1 <= n <= rows and 0 <= first and first + n <= total
        assert clip_of[first] == clip_of[first + n - 1], "a tile straddles two clips"
        assert (first - cu[clip_of[first]]) % rows == 0, "tiles start on the clip's own tile grid"
        cover[head, first:first + n] += 1
    assert np.all(cover == 1), "every (head, token) exactly once"
    # contiguous: head-major; dealt: all heads of one tile before the next; either way the clips of a
    # head come longest first (ties in packed order)
    heads_seen = [u[0] for u in live]
    if dealt:
        assert heads_seen == list(range(heads)) * n_tiles
        assert all(u[1:] == live[i - i % heads][1:] for i, u in enumerate(live))
        for c in range(len(lens)):      # no XCD has more tiles of a clip than another, but for one
            share = [0] * XCDS
            for i, u in enumerate(live):
                share[i % XCDS] += clip_of[u[1]] == c
            assert max(share) - min(share) <= 1
    else:
        assert heads_seen == sorted(heads_seen)
    for h in range(heads):
        clips = [int(clip_of[first]) for head, first, _ in live if head == h]
        runs = [c for i, c in enumerate(clips) if i == 0 or c != clips[i - 1]]
        assert len(runs) == len(set(runs)), "a clip's tiles are consecutive"
        want = sorted((c for c in range(len(lens)) if lens[c] > 0), key=lambda c: (-lens[c], c))
        assert runs == want
    return units


@pytest.mark.parametrize("rows", [128, 256])
def test_paper_workloads(rows):
    for name in ("C2", "C3", "C4"):
        wl = W.WORKLOADS[name]
        units = _check(wl.cu_seqlens, wl.n_heads, rows)
        live = int(np.sum(units[:, 0] >= 0))
        if name == "C4":       # 56,320 tokens: 220 tiles of 256 rows, 440 of 128, times 32 heads
            assert live == (56320 // rows) * 32
        if name == "C3":       # the block-diagonal schedule: tiles follow the clips, not total^2
            assert live == sum((n + rows - 1) // rows for n in wl.seqlens) * 24


@pytest.mark.parametrize("seed", range(12))
def test_random_clip_mixes(seed):
    rng = np.random.default_rng(seed)
    lens = [int(rng.integers(0, 3)) if rng.integers(0, 4) == 0 else int(rng.integers(1, 2000))
            for _ in range(int(rng.integers(1, 30)))]
    cu = np.concatenate([[0], np.cumsum(lens)])
    if cu[-1] == 0:
        lens[0] = 5
        cu = np.concatenate([[0], np.cumsum(lens)])
    _check(cu, int(rng.integers(1, 7)), int(rng.choice([32, 64, 128, 256])))


def test_unequal_clips_are_dealt_where_heads_do_not_divide_by_the_xcds():
    # 5,000 + 1,200 + 700 + 300 tokens: cut contiguously, every second XCD would hold 35 of the longest
    # clip's tiles of 12 heads and the others 25
    cu = np.cumsum([0, 300, 5000, 700, 1200])
    units = _check(cu, 12, 256)
    assert [int(u[0]) for u in units[:24]] == list(range(12)) * 2 and int(units[0][1]) == 300
    longest = [sum(1 for u in units[x::XCDS] if u[0] >= 0 and 300 <= u[1] < 5300) for x in range(XCDS)]
    assert longest == [30] * XCDS
    heads = [int(u[0]) for u in _units_in_order(_check(cu, 16, 256)) if u[0] >= 0]
    assert heads == sorted(heads)


@pytest.mark.parametrize("lens, heads, rows, dealt", [
    ((4096, 4095), 12, 256, False), ((4096, 4095), 13, 128, False), ((4096, 4095), 33, 256, False),
    ((8192, 8190, 8100), 33, 256, False),                        # nothing to even out, only heads to mix
    ((1500,) * 4 + (300,) * 8, 12, 256, False),                  # both orders need two rounds of long units
    ((1500,) * 4 + (300,) * 8, 4, 128, True),                    # two rounds against one
    ((5412, 440), 12, 256, True),                                # the second round is tiles of 36 rows, if dealt
    ((9000, 7000, 1100), 12, 256, True), ((4467, 490), 13, 256, True),
    ((700, 300), 12, 128, False),                                # one unit per CU at most
    ((20000, 15000), 13, 256, True), ((20000, 19900), 13, 256, False),
])
def test_units_are_dealt_where_the_contiguous_order_ends_later(lens, heads, rows, dealt):
    units = _check(np.concatenate([[0], np.cumsum(lens)]), heads, rows)
    assert (int(units[1][0]) == 1 and int(units[1][1]) == int(units[0][1])) == dealt


def test_equal_lengths_keep_packed_order_and_empty_input_has_no_workgroups():
    units = _check([0, 100, 200, 300], 1, 64)
    firsts = [int(u[1]) for u in _units_in_order(units) if u[0] >= 0]
    assert firsts == [0, 64, 100, 164, 200, 264]
    assert len(binding.vfm_schedule_units([0, 0, 0], 4, 256)) == 0


def test_more_clips_than_a_table_holds_are_scheduled_run_by_run():
    # 600 clips of 0..700 tokens: three launches (256 + 256 + 88 clips), whose grids follow one
    # another; each is a complete schedule of its own run of clips
    rng = np.random.default_rng(3)
    lens = rng.integers(0, 700, size=600)
    cu = np.concatenate([[0], np.cumsum(lens)])
    heads, rows = 3, 128
    units = binding.vfm_schedule_units(cu, heads, rows)
    at = 0
    for s0 in range(0, 600, 256):
        run = cu[s0:min(600, s0 + 256) + 1]
        n_tiles = int(sum((n + rows - 1) // rows for n in np.diff(run)))
        grid = XCDS * ((n_tiles * heads + XCDS - 1) // XCDS)
        _check(run, heads, rows, units[at:at + grid])
        at += grid
    assert at == len(units)


def test_forward_schedule_with_its_own_tile_height():
    # the forward cuts 128-row tiles when no clip of the launch has more than 1,024 tokens
    # (and always at head_dim 64), 256-row tiles otherwise
    for name, want in (("C2", 256), ("C4", 256)):
        wl = W.WORKLOADS[name]
        rows = binding.vfm_attn_fwd_tile_rows(wl.cu_seqlens, wl.head_dim)
        assert rows == want
        _check(wl.cu_seqlens, wl.n_heads, rows)
    images = np.arange(0, 289) * 256                        # 288 images of 256 tokens: two runs
    for run in (0, 1):
        assert binding.vfm_attn_fwd_tile_rows(images, 128, run) == 128
    spatial = W.WORKLOADS["C3"].spatial_cu_seqlens          # 36 frames of 256..1,024 tokens
    assert binding.vfm_attn_fwd_tile_rows(spatial, 128) == 128
    _check(spatial, 24, 128)
    assert binding.vfm_attn_fwd_tile_rows(W.WORKLOADS["C4"].cu_seqlens, 64) == 128


def test_argument_errors():
    lib = binding.load_library()
    import ctypes
    n = ctypes.c_int(0)
    cu = np.array([0, 10], dtype=np.int32)
    p = cu.ctypes.data_as(ctypes.POINTER(ctypes.c_int32))
    buf = np.zeros((8, 3), dtype=np.int32)
    pb = buf.ctypes.data_as(ctypes.POINTER(ctypes.c_int32))
    assert lib.vfm_schedule_units(None, 1, 10, 1, 256, pb, 8, ctypes.byref(n)) == 1      # NULL
    assert lib.vfm_schedule_units(p, 1, 10, 0, 256, pb, 8, ctypes.byref(n)) == 2         # no heads
    assert lib.vfm_schedule_units(p, 1, 10, 1, 0, pb, 8, ctypes.byref(n)) == 2           # no rows
    assert lib.vfm_schedule_units(p, 1, 11, 1, 256, pb, 8, ctypes.byref(n)) == 3         # cu vs total
    assert lib.vfm_schedule_units(p, 1, 10, 1, 256, pb, 4, ctypes.byref(n)) == 2 and n.value == 8   # too small
    assert lib.vfm_schedule_units(p, 1, 10, 1, 256, pb, 8, ctypes.byref(n)) == 0 and n.value == 8
    assert buf[0].tolist() == [0, 0, 10] and all(buf[i, 0] == -1 for i in range(1, 8))
