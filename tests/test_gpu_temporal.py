"""GPU parity of temporal attention (one sequence per pixel across a clip's frames) against the
fp64 oracle, through the C ABI."""
import numpy as np
import pytest

from oracle import vfm_oracle as orc
from paper_2503_12964_amd import workloads as W
from tests import parity_utils as U

pytestmark = pytest.mark.gpu


def _binding():
    from paper_2503_12964_amd import binding
    binding.load_library()
    return binding


CASES = {
    # frame counts 1, 2, 7, 16 and an empty clip; pixel counts that are not multiples of the 4 waves
    "t128": W.Workload("t128", ((16, 3, 5), (1, 2, 3), (0, 1, 1), (7, 1, 1), (2, 5, 5)), 3, 128, (32, 48, 48), seed=31),
    "t64": W.Workload("t64", ((5, 3, 3), (16, 1, 2), (3, 4, 1)), 2, 64, (16, 24, 24), seed=32),
    # more than 16 frames (the 32-row tile): 17, 24, 32 frames mixed with short clips, an empty one and
    # a single-frame one in the same call
    "t128_long": W.Workload("t128_long", ((17, 2, 3), (4, 3, 3), (32, 1, 5), (0, 1, 1), (24, 2, 2), (1, 3, 1)), 3, 128,
                            (32, 48, 48), seed=33),
    "t64_long": W.Workload("t64_long", ((32, 3, 1), (9, 2, 2), (20, 1, 1)), 2, 64, (16, 24, 24), seed=34),
}


def _check(wl, gpu, dev, heads=None):
    out, dq, dk, dv = gpu
    hs = slice(None) if heads is None else list(heads)
    host = {n: U.to_f64(t[:, hs, :]) for n, t in dev.items()}
    o_ref = orc.temporal_attn_fwd(host["q"], host["k"], host["v"], wl.thw, wl.cu_seqlens, wl.scale)
    g_ref = orc.temporal_attn_bwd(host["q"], host["k"], host["v"], host["dout"], wl.thw, wl.cu_seqlens, wl.scale)
    o = U.to_f64(out[:, hs, :])
    assert np.all(np.isfinite(o))
    # at most 32 keys: outputs are O(|v|), so the absolute bound is taken relative to max(1, |ref|)
    assert np.max(np.abs(o - o_ref) / np.maximum(1.0, np.abs(o_ref))) <= U.TOL_OUT_MAXABS
    assert U.rel_rms(o, o_ref) <= U.TOL_OUT_RELRMS
    U.assert_rows_close("out", o, o_ref, U.TOL_OUT_RELRMS)
    for nm, g, ref in zip(("dq", "dk", "dv"), (dq, dk, dv), g_ref):
        got = U.to_f64(g[:, hs, :])
        assert np.all(np.isfinite(got))
        r = U.rel_rms(got, ref)
        assert r <= U.TOL_GRAD_RELRMS, (nm, r)
        U.assert_rows_close(nm, got, ref, U.TOL_GRAD_RELRMS)       # every (token, head) row


def _run(b, wl):
    inp = W.make_inputs(wl)
    dev = {n: U.to_device(inp[n]) for n in ("q", "k", "v", "dout")}
    out = b.vfm_tattn_fwd(dev["q"], dev["k"], dev["v"], wl.thw, wl.cu_seqlens, wl.scale)
    dq, dk, dv = b.vfm_tattn_bwd(dev["q"], dev["k"], dev["v"], dev["dout"], wl.thw, wl.cu_seqlens, wl.scale)
    return dev, (out, dq, dk, dv)


@pytest.mark.parametrize("name", list(CASES))
def test_temporal_attention_matches_oracle(name):
    wl = CASES[name]
    dev, gpu = _run(_binding(), wl)
    _check(wl, gpu, dev)


def test_single_frame_clip_copies_values_and_has_zero_qk_gradients():
    wl = CASES["t128"]
    dev, (out, dq, dk, dv) = _run(_binding(), wl)
    a, b = int(wl.cu_seqlens[1]), int(wl.cu_seqlens[2])      # the (1,2,3) clip
    assert np.array_equal(U.to_bits(out[a:b]), U.to_bits(dev["v"][a:b]))
    assert not np.any(U.to_f64(dq[a:b])) and not np.any(U.to_f64(dk[a:b]))
    assert np.array_equal(U.to_bits(dv[a:b]), U.to_bits(dev["dout"][a:b]))


LONG = {
    # more than 32 frames (Section 4.6: videos of hundreds of frames).  Up to 128, a workgroup per sequence: 33,
    # 48, 121 frames, block multiples (64, 96) and short clips, an empty and a single-frame one in the call
    "t128_33_48": W.Workload("t128_33_48", ((33, 2, 3), (48, 1, 5), (4, 3, 3), (0, 1, 1), (1, 2, 2), (64, 1, 2)), 3, 128,
                             (32, 48, 48), seed=35),
    "t128_121": W.Workload("t128_121", ((121, 3, 2), (96, 1, 1), (17, 2, 2)), 2, 128, (32, 48, 48), seed=36),
    "t64_long": W.Workload("t64_100", ((100, 2, 2), (33, 1, 3), (65, 1, 1), (2, 2, 2)), 2, 64, (16, 24, 24), seed=37),
    "t128_300": W.Workload("t128_300", ((300, 1, 2),), 1, 128, (32, 48, 48), seed=38),
    # more than 128, a wavefront per 32-row block: block multiples and both sides of one, several long clips, and
    # short, empty and single-frame ones, few enough to be walked in blocks with them
    "t128_129_200": W.Workload("t128_129_200", ((129, 2, 3), (200, 1, 2), (0, 1, 1), (1, 2, 2), (160, 1, 3), (17, 1, 2), (100, 1, 1)),
                               2, 128, (32, 48, 48), seed=39),
    "t64_161_300": W.Workload("t64_161_300", ((161, 1, 3), (1, 1, 1), (300, 2, 1), (0, 2, 2), (64, 1, 2), (9, 2, 2)), 3, 64,
                              (16, 24, 24), seed=40),
}


@pytest.mark.parametrize("name", list(LONG))
def test_more_than_thirty_two_frames(name):
    wl = LONG[name]
    dev, gpu = _run(_binding(), wl)
    _check(wl, gpu, dev)


@pytest.mark.parametrize("name", ["t128_33_48", "t128_129_200", "t64_161_300"])
def test_long_clip_statistics_do_not_leak_into_dq(name):
    # with more than 128 frames the dq rows carry the queries' statistics while the call runs; afterwards
    # every dq element is a gradient, also after a second call into the same buffers.  (Up to 128 frames
    # the statistics are in LDS: buffers full of NaN must not matter there either.)
    import torch
    wl = LONG[name]
    b = _binding()
    inp = W.make_inputs(wl)
    dev = {n: U.to_device(inp[n]) for n in ("q", "k", "v", "dout")}
    dq, dk, dv = (torch.full_like(dev["q"], float("nan")) for _ in range(3))
    for _ in range(2):
        b.vfm_tattn_bwd(dev["q"], dev["k"], dev["v"], dev["dout"], wl.thw, wl.cu_seqlens, wl.scale, dq=dq, dk=dk, dv=dv)
    host = {n: U.to_f64(t) for n, t in dev.items()}
    g_ref = orc.temporal_attn_bwd(host["q"], host["k"], host["v"], host["dout"], wl.thw, wl.cu_seqlens, wl.scale)
    for nm, g, ref in zip(("dq", "dk", "dv"), (dq, dk, dv), g_ref):
        assert U.rel_rms(U.to_f64(g), ref) <= U.TOL_GRAD_RELRMS, nm
        U.assert_rows_close(nm, U.to_f64(g), ref, U.TOL_GRAD_RELRMS)


def test_single_frame_clip_in_a_long_call():
    # a few single frames beside clips of up to 32 frames are served by the latter's kernels
    wl = CASES["t128_long"]
    dev, (out, dq, dk, dv) = _run(_binding(), wl)
    a, b = int(wl.cu_seqlens[5]), int(wl.cu_seqlens[6])      # the (1,3,1) clip
    assert np.array_equal(U.to_bits(out[a:b]), U.to_bits(dev["v"][a:b]))
    assert not np.any(U.to_f64(dq[a:b])) and not np.any(U.to_f64(dk[a:b]))
    assert np.array_equal(U.to_bits(dv[a:b]), U.to_bits(dev["dout"][a:b]))


def test_full_size_c4_every_element():
    """The 56,320-token latent (16 frames x 3,520 pixels), 32 heads: every element of out, dq,
    dk, dv against the oracle, four heads at a time."""
    wl = W.WORKLOADS["C4"]
    dev, gpu = _run(_binding(), wl)
    for h0 in range(0, wl.n_heads, 4):
        _check(wl, gpu, dev, heads=range(h0, h0 + 4))


@pytest.mark.parametrize("frames", [17, 32, 33, 64, 65, 96, 97, 128, 129])
@pytest.mark.parametrize("head_dim", [64, 128])
def test_block_edges(frames, head_dim):
    # the workgroup-per-sequence kernels hold 1 to 4 blocks of 32 frames: both ends of every size, the
    # first length past them, and a short clip in the same call
    wl = W.Workload(f"edge{frames}", ((frames, 1, 3), (5, 2, 1)), 2, head_dim, (0, head_dim // 2, head_dim // 2), seed=frames)
    dev, gpu = _run(_binding(), wl)
    _check(wl, gpu, dev)


@pytest.mark.parametrize("head_dim", [64, 128])
def test_clips_take_the_kernels_of_their_own_frame_count(head_dim):
    """A call that holds every class of frame counts, each with more sequences than join a longer class: a clip's
    results are to the bit what a call of its own gives.  One class is spread over two clips around an
    empty one."""
    import torch
    frames = (5, 100, 1, 17, 0, 200, 70, 16, 40, 129, 32)
    wl = W.Workload("classes", tuple((t, 29, 30) for t in frames), 12, head_dim, (0, head_dim // 2, head_dim // 2), seed=51)
    b = _binding()
    gen = torch.Generator(device="cuda").manual_seed(51)
    dev = {n: torch.empty((wl.total_tokens, 12, head_dim), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
           for n in ("q", "k", "v", "dout")}

    def both_ways(x, thw, cu):
        return (b.vfm_tattn_fwd(x["q"], x["k"], x["v"], thw, cu, wl.scale),
                *b.vfm_tattn_bwd(x["q"], x["k"], x["v"], x["dout"], thw, cu, wl.scale))

    gpu = both_ways(dev, wl.thw, wl.cu_seqlens)
    for i in range(len(frames)):
        lo, hi = int(wl.cu_seqlens[i]), int(wl.cu_seqlens[i + 1])
        if lo == hi:
            continue
        alone = both_ways({n: t[lo:hi].contiguous() for n, t in dev.items()}, wl.thw[i:i + 1], [0, hi - lo])
        for nm, x, y in zip(("out", "dq", "dk", "dv"), gpu, alone):
            assert torch.equal(x[lo:hi].view(torch.int16), y.view(torch.int16)), (nm, frames[i])


@pytest.mark.parametrize("head_dim", [64, 128])
def test_few_short_clips_join_longer_ones(head_dim):
    # every class of frame counts in one small call: all of them end in the kernels of the longest
    wl = W.Workload("few", tuple((t, 1, 2 + i % 3) for i, t in enumerate((5, 100, 1, 17, 0, 200, 70, 16, 40, 129, 32))), 3,
                    head_dim, (0, head_dim // 2, head_dim // 2), seed=52)
    dev, gpu = _run(_binding(), wl)
    _check(wl, gpu, dev)


def test_many_pixels_beside_a_long_clip():
    """262,144 single-frame pixels and 32 heads beside one 100-frame clip: 2^23 sequences, which at a workgroup
    of the long clip's size each would be more threads than a launch can have.  Single frames copy v
    and dout to the bit (P is within a few fp32 ulp of 1); dS = P (dP - P dP) is within 2^-21 |dP| of 0, and
    with |dP| < 100, |q|, |k| < 8 and the scale 1/11 so are the gradients of q and k within 4e-5."""
    import torch
    b = _binding()
    n, t, heads, hd = 512 * 512, 100, 32, 128
    thw = np.array([[1, 512, 512], [t, 1, 1]], dtype=np.int32)
    cu = [0, n, n + t]
    gen = torch.Generator(device="cuda").manual_seed(5)
    q, k, v, do = (torch.empty((n + t, heads, hd), dtype=torch.bfloat16, device="cuda").normal_(generator=gen) for _ in range(4))
    out = b.vfm_tattn_fwd(q, k, v, thw, cu, hd ** -0.5)
    dq, dk, dv = b.vfm_tattn_bwd(q, k, v, do, thw, cu, hd ** -0.5)
    assert torch.equal(out[:n], v[:n]) and torch.equal(dv[:n], do[:n])
    assert dq[:n].abs().max() <= 4e-5 and dk[:n].abs().max() <= 4e-5
    wl = W.Workload("tail", ((t, 1, 1),), heads, hd, (0, 64, 64), seed=0)
    tail = {name: x[n:].contiguous() for name, x in (("q", q), ("k", k), ("v", v), ("dout", do))}
    _check(wl, tuple(x[n:].contiguous() for x in (out, dq, dk, dv)), tail)


@pytest.mark.parametrize("frames", [64, 128])
def test_probabilities_are_rounded_against_a_running_maximum(frames):
    """Key blocks of 32 are taken in turn, P relative to the largest score so far, so that every new maximum is
    exactly 1 in bf16.  Done in 64 bits with only that rounding (and out's) this is the distance from
    the exact result that the call may have: P relative to the row's maximum is 1.6 to 2.4% further
    off.  0.5% covers the scatter of the norm over 3 million elements (1e-3) and fp32 sums (1e-7)."""
    wl = W.Workload("reference", ((frames, 1, 12800 // frames),), 2, 128, (0, 64, 64), seed=53)
    b = _binding()
    inp = W.make_inputs(wl)
    out = U.to_f64(b.vfm_tattn_fwd(*(U.to_device(inp[n]) for n in ("q", "k", "v")), wl.thw, wl.cu_seqlens, wl.scale))
    q, k, v = (U.bits_to_f64(inp[n]).reshape(frames, -1, 2, 128).transpose(1, 2, 0, 3) for n in ("q", "k", "v"))
    s = (q @ k.swapaxes(-1, -2)) * wl.scale
    p = np.exp(s - s.max(-1, keepdims=True))
    exact = p @ v / p.sum(-1, keepdims=True)

    def bf16(x):
        return W.bf16_bits_to_f32(W.f32_to_bf16_bits(x.astype(np.float32))).astype(np.float64)

    m, l, acc = np.full(s.shape[:3] + (1,), -np.inf), 0.0, 0.0
    for j in range(0, frames, 32):
        m_new = np.maximum(m, s[..., j:j + 32].max(-1, keepdims=True))
        p = np.exp(s[..., j:j + 32] - m_new)
        alpha = np.exp(m - m_new)
        l, acc, m = l * alpha + p.sum(-1, keepdims=True), acc * alpha + bf16(p) @ v[..., j:j + 32, :], m_new
    may = np.linalg.norm(bf16(acc / l) - exact)
    got = out.reshape(frames, -1, 2, 128).transpose(1, 2, 0, 3)
    assert np.linalg.norm(got - exact) <= 1.005 * may
