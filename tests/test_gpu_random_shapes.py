"""Randomised packed shapes: many clips of arbitrary lengths (including empty and one-token
clips, lengths around every tile size), odd head counts, both head dims; the whole
rope -> forward -> backward path against the oracle."""
import numpy as np
import pytest

from paper_2503_12964_amd import workloads as W
from tests import parity_utils as U
from tests.test_gpu_parity import _assert_parity, _run_fwd_bwd

pytestmark = pytest.mark.gpu


def _random_workload(seed):
    rng = np.random.default_rng(seed)
    hd = (64, 128)[seed % 2]
    heads = int(rng.choice([1, 3, 5]))
    n_clips = int(rng.integers(3, 40))
    grids = []
    for _ in range(n_clips):
        kind = rng.integers(0, 6)
        if kind == 0:
            grids.append((0, 1, 1))                               # empty clip
        elif kind == 1:
            grids.append((1, 1, 1))                               # one token
        elif kind == 2:                                           # around a tile boundary
            n = int(rng.choice([31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257]))
            grids.append((1, 1, n))
        else:
            grids.append((int(rng.integers(1, 5)), int(rng.integers(1, 13)), int(rng.integers(1, 13))))
    dims = (16, 24, 24) if hd == 64 else (32, 48, 48)
    return W.Workload(f"rand{seed}", tuple(grids), heads, hd, dims, seed=100 + seed)


@pytest.mark.parametrize("seed", range(8))
def test_random_packed_shapes(seed):
    wl = _random_workload(seed)
    if wl.total_tokens == 0:
        pytest.skip("all clips empty")
    gpu, host = _run_fwd_bwd(wl, rope=True)
    # short clips make outputs O(|v|): bound the absolute error relative to max(1, |ref|)
    _assert_parity(wl, gpu, host, relative_maxabs=True)


def _random_long_workload(seed):
    """A few clips of arbitrary length up to 6,000 tokens (many ring turns and every remainder of
    the unrolled loops), some of them empty, tiny, or a token or two around a tile multiple."""
    rng = np.random.default_rng(1000 + seed)
    hd = 128 if seed % 4 else 64
    grids = []
    for _ in range(int(rng.integers(1, 12))):
        kind = rng.integers(0, 5)
        if kind == 0:
            n = int(rng.integers(0, 3))
        elif kind == 1:
            n = int(rng.choice([32, 64, 96, 128, 192, 256, 384, 512, 768, 1024])) + int(rng.integers(-2, 3))
        else:
            n = int(rng.integers(1, 6000))
        grids.append((1, 1, n) if n else (0, 1, 1))
    dims = (16, 24, 24) if hd == 64 else (32, 48, 48)
    return W.Workload(f"long{seed}", tuple(grids), int(rng.choice([1, 2, 3])), hd, dims, seed=5000 + seed)


@pytest.mark.parametrize("seed", [201, 203, 228, 237])
def test_random_long_clips(seed):
    wl = _random_long_workload(seed)
    gpu, host = _run_fwd_bwd(wl, rope=True)
    _assert_parity(wl, gpu, host, relative_maxabs=True)


def test_maximum_number_of_clips():
    # 256 clips (the table's capacity) of 1..40 tokens
    rng = np.random.default_rng(7)
    grids = tuple((1, 1, int(n)) for n in rng.integers(1, 41, size=256))
    wl = W.Workload("max_clips", grids, 2, 128, (32, 48, 48), seed=77)
    gpu, host = _run_fwd_bwd(wl, rope=True)
    _assert_parity(wl, gpu, host, relative_maxabs=True)


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("lengths", [
    (64, 63, 33, 32, 31, 2, 1),                       # up to 64: any number of clips takes the one pass
    (128, 127, 97, 96, 65, 64, 40, 20, 1),            # four wavefronts, 128 keys
    (256, 255, 225, 224, 193, 161, 160, 129, 128, 33, 16, 5),   # eight wavefronts, odd and even block counts
], ids=["64", "128", "256"])
def test_one_pass_backward_block_edges(head_dim, lengths):
    """Clips of at most 256 tokens whose backward is one workgroup per (clip, head): every remainder
    of the 32-row blocks, enough (clip, head) units (over 128 and over 256/3) to leave the two-pass kernels."""
    grids = tuple((1, 1, n) for n in lengths for _ in range(3)) + ((0, 1, 1),)
    dims = (16, 24, 24) if head_dim == 64 else (32, 48, 48)
    wl = W.Workload(f"one_pass{lengths[0]}", grids, 5, head_dim, dims, seed=300 + lengths[0])
    gpu, host = _run_fwd_bwd(wl)
    _assert_parity(wl, gpu, host, relative_maxabs=True)


@pytest.mark.parametrize("lengths", [(257, 127), (383, 384, 385, 64), (640, 513, 33, 1)], ids=["257", "384", "640"])
def test_two_pass_tile_edges_head_dim_64(lengths):
    """Head_dim 64 beyond the one pass: 128-row query and key tiles with every kind of remainder (a row, a row
    short, wavefronts without a row)."""
    wl = W.Workload(f"d64_{lengths[0]}", tuple((1, 1, n) for n in lengths), 3, 64, (16, 24, 24), seed=640 + lengths[0])
    gpu, host = _run_fwd_bwd(wl)
    _assert_parity(wl, gpu, host, relative_maxabs=True)


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("heads, lens, dealt_rows", [(2, (1301, 700, 700, 257, 5), ()), (12, (1301, 700, 700, 257, 5), (128,)),
                                                     (12, (5000, 1200, 700, 300), (128, 256)), (13, (4467, 490), (256,))], ids=str)
def test_dealt_units_of_unequal_clips(heads, lens, dealt_rows, head_dim):
    """Heads that do not divide by the XCDs and clips of unequal length: whether the tiles of a pass (of 128 or 256
    rows) are dealt out or not, each clip gets the bits that it gets in a call of its own."""
    import torch
    from paper_2503_12964_amd import binding as b
    for rows in (128, 256):      # dealt: the second workgroup has the first tile's next head
        second = b.vfm_schedule_units(np.concatenate([[0], np.cumsum(lens)]), heads, rows)[1].tolist()
        assert (second == [1, 0, rows]) == (rows in dealt_rows)
    n = sum(lens)
    gen = torch.Generator(device="cuda").manual_seed(heads + head_dim)
    q, k, v, do = (torch.empty((n, heads, head_dim), device="cuda").normal_(generator=gen).to(torch.bfloat16) for _ in range(4))

    def run(lo, hi, cu):
        x = [t[lo:hi].contiguous() for t in (q, k, v, do)]
        out, lse = b.vfm_attn_fwd(*x[:3], cu, 0.125)
        return [out, lse.t().contiguous(), *b.vfm_attn_bwd(*x[:3], out, lse, x[3], cu, 0.125)]

    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    whole = run(0, n, cu)
    for lo, hi in zip(cu, cu[1:]):
        for got, alone in zip(whole, run(lo, hi, np.asarray([0, hi - lo], dtype=np.int32))):
            assert torch.equal(got[lo:hi].view(torch.uint8), alone.view(torch.uint8))


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("lengths", [(64, 63, 33, 32, 31, 17, 5, 2, 1), (128, 127, 97, 65, 32, 16),
                                     (256, 255, 225, 193, 160, 129, 33, 8)], ids=["64", "128", "256"])
def test_a_clip_does_not_depend_on_its_pack_mates(head_dim, lengths):
    """Clips of at most 256 tokens take the one pass or the two-pass kernels by what else is in the run, and
    equal ranges may come through the cross-attention entry: every route gives the same bits."""
    import torch
    from paper_2503_12964_amd import binding as b
    lens, heads = lengths * 6, 4        # 144 units and more: the one pass
    n = sum(lens)
    gen = torch.Generator(device="cuda").manual_seed(head_dim + lengths[0])
    x = [torch.empty((n + 1100, heads, head_dim), device="cuda").normal_(generator=gen).to(torch.bfloat16) for _ in range(4)]

    def run(lo, hi, cu, cross=False):
        q, k, v, do = (t[lo:hi].contiguous() for t in x)
        cu = np.asarray(cu, dtype=np.int32)
        scale = head_dim ** -0.5
        fwd = b.vfm_xattn_fwd(q, k, v, cu, cu, scale) if cross else b.vfm_attn_fwd(q, k, v, cu, scale)
        bwd = b.vfm_xattn_bwd(q, k, v, *fwd, do, cu, cu, scale) if cross else b.vfm_attn_bwd(q, k, v, *fwd, do, cu, scale)
        return [fwd[0], fwd[1].T.contiguous(), *bwd]

    cu = np.concatenate([[0], np.cumsum(lens)])
    want = run(0, n, cu)
    routes = {"beside 1,100 tokens": (0, n, run(0, n + 1100, [*cu, n + 1100])), "cross": (0, n, run(0, n, cu, cross=True))}
    for i in range(len(lengths)):
        lo, hi = int(cu[i]), int(cu[i + 1])
        routes[f"alone {lens[i]}"] = (lo, hi, run(lo, hi, [0, hi - lo]))
    for route, (lo, hi, got) in routes.items():
        for nm, g, w in zip(("out", "lse", "dq", "dk", "dv"), got, want):
            assert torch.equal(g[:hi - lo], w[lo:hi]), (route, nm)


def test_one_pass_backward_under_graph_replay_and_without_workspace():
    """The one pass ignores the statistics buffers: both entry points give the same bits, and a
    captured call gives them again on every replay."""
    import torch
    from paper_2503_12964_amd import binding as b
    wl = W.Workload("one_pass_graph", tuple((1, 1, n) for n in (200, 256, 129) * 10), 4, 128, (32, 48, 48), seed=9)
    q, k, v, do = (U.to_device(W.make_inputs(wl)[n]) for n in ("q", "k", "v", "dout"))
    out, lse = b.vfm_attn_fwd(q, k, v, wl.cu_seqlens, wl.scale)
    want = b.vfm_attn_bwd(q, k, v, out, lse, do, wl.cu_seqlens, wl.scale)
    got = [torch.empty_like(q) for _ in range(3)]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        b.vfm_attn_bwd_noalloc(q, k, v, out, lse, do, wl.cu_seqlens, wl.scale, *got)
    for _ in range(3):
        for t in got:
            t.fill_(7.0)
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a.view(torch.int16), c.view(torch.int16)) for a, c in zip(got, want))


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("lengths", [(1100, 700, 20, 1), (1025, 257, 33)], ids=["few_keys", "tails"])
def test_statistics_from_the_dq_pass(lengths, head_dim):
    """Packs with a clip of more than 1,024 tokens (at head_dim 64: more than 256): the dQ pass forms Delta (not
    that of clips of at most 32 keys) and the dK/dV pass reads it; with dq written over dout both come from
    the separate pass and the gradients are the same bits."""
    import torch
    from paper_2503_12964_amd import binding as b
    dims = (16, 24, 24) if head_dim == 64 else (32, 48, 48)
    wl = W.Workload("dq_first", tuple((1, 1, n) for n in lengths), 3, head_dim, dims, seed=31)
    gpu, host = _run_fwd_bwd(wl)
    _assert_parity(wl, gpu, host, relative_maxabs=True)
    q, k, v, do = (U.to_device(W.make_inputs(wl)[n]) for n in ("q", "k", "v", "dout"))
    got = b.vfm_attn_bwd(q, k, v, gpu[0], gpu[1], do, wl.cu_seqlens, wl.scale, dq=do)
    assert all(torch.equal(x.view(torch.int16), y.view(torch.int16)) for x, y in zip(got, gpu[2:]))


@pytest.mark.parametrize("cross", [False, True], ids=["self", "cross"])
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("lengths,heads", [((1000, 700, 300, 20), 3), ((256, 129, 31), 2), ((200, 64, 256, 7) * 20, 3), ((1300, 40), 2)],
                         ids=["one_grid", "few_short", "one_pass", "two_passes"])
def test_dq_in_place_of_q_or_dout(lengths, heads, head_dim, cross):
    """dq may be the buffer of q or of dout: the rows that a workgroup overwrites with dq are read by every
    dK/dV workgroup of the sequence, so the two must not run side by side.  Same bits as without."""
    import torch
    from paper_2503_12964_amd import binding as b
    cu = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    gen = torch.Generator(device="cuda").manual_seed(int(cu[-1]))
    q, k, v, do = (torch.empty((int(cu[-1]), heads, head_dim), device="cuda").normal_(generator=gen).to(torch.bfloat16)
                   for _ in range(4))
    scale = head_dim ** -0.5
    out, lse = b.vfm_attn_fwd(q, k, v, cu, scale)

    def bwd(qq, dd, dq):
        if cross:
            return b.vfm_xattn_bwd(qq, k, v, out, lse, dd, cu, cu, scale, dq=dq)
        return b.vfm_attn_bwd(qq, k, v, out, lse, dd, cu, scale, dq=dq)

    want = bwd(q, do, None)
    for over in ("q", "dout"):
        qq, dd = q.clone(), do.clone()
        got = bwd(qq, dd, qq if over == "q" else dd)
        names = ("dq", "dk", "dv")
        if cross and max(lengths) >= 1024:      # split queries: dk, dv are summed with atomics
            names = ("dq",)
        for nm, g, w in zip(names, got, want):
            assert torch.equal(g, w), (over, nm)
