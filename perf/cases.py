"""The work this library is used for, as timed cases: what one layer of a video diffusion
transformer asks of it, through the calls of paper_2503_12964_amd.binding.

A case names one of four paths:

  self      position encoding of q and k (plain RoPE, or per-head normalisation fused with
            it), full attention over packed clips, and in training its backward and the
            backward of the position encoding; optionally with one sequence per latent frame
            (the spatial half of a spatial-temporal transformer)
  cross     video queries against text keys and values, forward and in training backward
  temporal  one sequence per pixel across a clip's frames, forward and in training backward
  fp8       inference on 8-bit operands: RoPE, packing, forward

Grids are texts such as "2x16x16,40*1x32x32" (frames x height x width of a latent clip, with
an optional count), prompts likewise ("226,77").  Training passes let the calls allocate their
results, as an autograd function does; inference passes reuse the buffers of the last step.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2503_12964_amd import binding as vfm

THETA = 10000.0
EPS = 1e-6


def _case(name, path, grids, heads, head_dim, train, **more):
    case = {"path": path, "grids": grids, "heads": heads, "head_dim": head_dim, "train": train}
    if name:
        case["name"] = name
    case.update(more)
    return case


def listed():
    return [
        # the smallest call: one 32-token clip, two narrow heads; launches and host work are all of it
        _case("tiny_step", "self", "1*2x4x4", 2, 64, True, encode="rope", spatial=False, builtin_scratch=False),
        # sampling small pictures with classifier-free guidance: batch of two 256-token images, forward only
        _case("image_pair_denoise", "self", "2*1x16x16", 32, 128, False, encode="rope", spatial=False, builtin_scratch=False),
        # clips of odd shapes at head_dim 64 (tails everywhere), trained without a workspace of the caller's
        _case("ragged_step_d64", "self", "3x17x23,1x15x9,5x13x31,2x29x37,7x11x5,1x33x33", 12, 64, True, encode="rope", spatial=False, builtin_scratch=True),
        # 256px-class training: two clips of 4,096 tokens, normalised q and k
        _case("two_clip_step", "self", "2*4x32x32", 16, 128, True, encode="qknorm", spatial=False, builtin_scratch=False),
        # eight clips of different shapes packed into one 28,704-token sequence
        _case("mixed_pack_step", "self", "2x16x16,4x24x40,8x32x32,3x22x40,6x16x16,5x24x40,1x32x32,7x22x40", 24, 128, True, encode="qknorm", spatial=False, builtin_scratch=False),
        # image pre-training: a 73,728-token context filled with 256-token images
        _case("image_pack_step", "self", "288*1x16x16", 32, 128, True, encode="rope", spatial=False, builtin_scratch=False),
        # spatial half of a spatial-temporal transformer on a 720p-class latent: 16 frames of 3,520 tokens
        _case("spatial_step", "self", "1*16x44x80", 32, 128, True, encode="rope", spatial=True, builtin_scratch=False),
        # full attention over the same latent, 56,320 tokens: the headline workload and the largest
        _case("long_clip_step", "self", "1*16x44x80", 32, 128, True, encode="rope", spatial=False, builtin_scratch=False),
        # cross-attention of that latent to a 512-token text embedding
        _case("text_cross_step", "cross", "1*16x44x80", 32, 128, True, prompts="512"),
        # temporal half: 16 latent frames (a 121-frame video)
        _case("temporal_step", "temporal", "1*16x44x80", 32, 128, True),
        # temporal half on a longer video: 64 latent frames, 8 heads
        _case("long_temporal_step", "temporal", "1*64x44x80", 8, 128, True),
        # 8-bit inference over the 720p-class latent
        _case("fp8_denoise", "fp8", "1*16x44x80", 32, 128, False),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid(rng, max_frames, max_side):
    return "%dx%dx%d" % (_log_uniform(rng, 1, max_frames), rng.randint(4, max_side), rng.randint(4, max_side))


def draw(rng):
    kind = rng.choice(["clips", "clips", "images", "spatial", "denoise", "cross", "temporal", "fp8"])
    head_dim = 128 if rng.random() < 0.75 else 64
    if kind == "clips":        # training on a few clips of any shape, 100 to about 20,000 tokens
        grids = []
        while not grids or (len(grids) < 8 and rng.random() < 0.6):
            grids.append(_grid(rng, 8, 48))
        while sum(_lengths(",".join(grids))) > 24000:
            grids.pop() if len(grids) > 1 else grids.__setitem__(0, _grid(rng, 8, 48))
        return _case(None, "self", ",".join(grids), rng.choice([2, 4, 8, 12, 16, 24, 32]), head_dim, True,
                     encode=rng.choice(["rope", "qknorm"]), spatial=False, builtin_scratch=rng.random() < 0.25)
    if kind == "images":       # packs of images of one class of sizes, up to the 73,728-token context
        h, w = rng.randint(8, 32), rng.randint(8, 32)
        n = max(2, min(_log_uniform(rng, 8, 512), 73728 // (h * w)))
        first = max(1, n // 2)
        grids = "%d*1x%dx%d" % (first, h, w) + (",%d*1x%dx%d" % (n - first, w, max(8, h - rng.randint(0, 7))) if n > first else "")
        return _case(None, "self", grids, rng.choice([8, 16, 24, 32]), head_dim, True,
                     encode=rng.choice(["rope", "qknorm"]), spatial=False, builtin_scratch=False)
    if kind == "spatial":      # one sequence per latent frame
        return _case(None, "self", "1*%dx%dx%d" % (rng.randint(4, 20), rng.randint(12, 48), rng.randint(12, 80)),
                     rng.choice([8, 16, 24]), head_dim, True, encode="rope", spatial=True, builtin_scratch=False)
    if kind == "denoise":      # sampling: one clip or a guided pair, from a thumbnail to a long clip
        return _case(None, "self", "%d*%s" % (rng.randint(1, 2), _grid(rng, 12, 48)), rng.choice([8, 16, 24, 32]), head_dim,
                     False, encode=rng.choice(["rope", "qknorm"]), spatial=False, builtin_scratch=False)
    if kind == "cross":        # one to three clips, each with a prompt of its own length
        n = rng.randint(1, 3)
        grids = ",".join(_grid(rng, 12, 48) for _ in range(n))
        prompts = ",".join(str(_log_uniform(rng, 16, 512)) for _ in range(n))
        return _case(None, "cross", grids, rng.choice([8, 16, 24, 32]), head_dim, rng.random() < 0.75, prompts=prompts)
    if kind == "temporal":     # a few frames up to a few hundred
        frames, side = _log_uniform(rng, 4, 200), rng.randint(8, 48)
        heads = rng.choice([4, 8, 16])
        while frames * side * side * heads > 2_000_000:
            side -= 1
        return _case(None, "temporal", "1*%dx%dx%d" % (frames, side, side + rng.randint(0, 5)), heads, head_dim, rng.random() < 0.75)
    return _case(None, "fp8", "%d*%s" % (rng.randint(1, 2), _grid(rng, 16, 64)), rng.choice([8, 16, 32]), head_dim, False)


# ---------------------------------------------------------------- shapes
def _grids(text):
    out = []
    for part in text.split(","):
        n, _, shape = part.rpartition("*")
        out += [tuple(int(x) for x in shape.split("x"))] * int(n or 1)
    return out


def _lengths(text):
    return [t * h * w for t, h, w in _grids(text)]


def _prefix(lens):
    return np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)


def _sequences(case):
    """Query and key lengths of every attention sequence of a self or cross case."""
    grids = _grids(case["grids"])
    if case.get("spatial"):
        lens = [h * w for t, h, w in grids for _ in range(t)]
    else:
        lens = [t * h * w for t, h, w in grids]
    if case["path"] == "cross":
        return lens, [int(x) for x in case["prompts"].split(",")]
    return lens, lens


def _axis_split(head_dim):
    return (head_dim // 4, 3 * head_dim // 8, 3 * head_dim // 8)


# ---------------------------------------------------------------- one case
def prepare(case, seed):
    """Unit-variance bf16 activations (what normalised queries and keys have) and the buffers a
    program keeps between steps."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(int(seed))
    heads, hd, path = case["heads"], case["head_dim"], case["path"]
    grids = _grids(case["grids"])
    total = sum(t * h * w for t, h, w in grids)

    def normal(rows):
        return torch.randn((rows, heads, hd), generator=gen, device=dev, dtype=torch.float32).to(torch.bfloat16)

    lens_q, lens_k = _sequences(case)
    rows_k = sum(lens_k) if path == "cross" else total
    s = {"case": case, "scale": 1.0 / math.sqrt(hd), "dims": _axis_split(hd),
         "thw": np.asarray(grids, dtype=np.int32).reshape(-1, 3), "clips": _prefix([t * h * w for t, h, w in grids]),
         "cu_q": _prefix(lens_q), "cu_k": _prefix(lens_k),
         "q": normal(total), "k": normal(rows_k), "v": normal(rows_k)}
    if case["train"]:
        s["dout"] = normal(total)
    if case.get("encode") == "qknorm":
        gains = 1.0 + 0.25 * torch.randn((2, hd), generator=gen, device=dev, dtype=torch.float32)
        s["gain_q"], s["gain_k"] = gains[0].contiguous(), gains[1].contiguous()
        s["yq"], s["yk"] = torch.empty_like(s["q"]), torch.empty_like(s["k"])
    if path in ("self", "cross") and case["train"]:
        if path == "cross":
            need = vfm.vfm_xattn_bwd_workspace_size(total, rows_k, heads, hd)
        else:
            need = vfm.vfm_attn_bwd_workspace_size(total, heads, hd)
        s["workspace"] = torch.empty(max(need, 256), dtype=torch.uint8, device=dev)
    if not case["train"]:
        s["out"] = torch.empty_like(s["q"])
        s["lse"] = torch.empty((heads, total), dtype=torch.float32, device=dev)
    if path == "fp8":
        sizes = vfm.vfm_fp8_pack_sizes(s["clips"], heads, hd)
        s["packed"] = [torch.empty(max(n, 16), dtype=torch.uint8, device=dev) for n in sizes]
    return s


def _encode(s):
    """q and k as attention takes them.  Plain RoPE works in place (a further pass turns them
    further: still unit-variance draws); the normalised form writes buffers of its own."""
    thw, cu, dims = s["thw"], s["clips"], s["dims"]
    if s["case"].get("encode") == "qknorm":
        return (vfm.vfm_qknorm_rope3d(s["q"], s["gain_q"], EPS, thw, cu, dims, THETA, y=s["yq"]),
                vfm.vfm_qknorm_rope3d(s["k"], s["gain_k"], EPS, thw, cu, dims, THETA, y=s["yk"]))
    return vfm.vfm_rope3d(s["q"], thw, cu, dims, THETA), vfm.vfm_rope3d(s["k"], thw, cu, dims, THETA)


def _run_self(s):
    case, cu, scale = s["case"], s["cu_q"], s["scale"]
    q, k = _encode(s)
    if not case["train"]:
        out, lse = vfm.vfm_attn_fwd(q, k, s["v"], cu, scale, out=s["out"], lse=s["lse"])
        return {"q": q, "k": k, "out": out, "lse": lse}
    out, lse = vfm.vfm_attn_fwd(q, k, s["v"], cu, scale)
    if case["builtin_scratch"]:
        dq, dk, dv = torch.empty_like(q), torch.empty_like(k), torch.empty_like(s["v"])
        vfm.vfm_attn_bwd_noalloc(q, k, s["v"], out, lse, s["dout"], cu, scale, dq, dk, dv)
    else:
        dq, dk, dv = vfm.vfm_attn_bwd(q, k, s["v"], out, lse, s["dout"], cu, scale, workspace=s["workspace"])
    got = {"out": out, "lse": lse, "dv": dv}
    if case["encode"] == "qknorm":
        for n, x, dy in (("q", s["q"], dq), ("k", s["k"], dk)):
            got["d" + n], got["dgain_" + n] = vfm.vfm_qknorm_rope3d_bwd(
                x, s["gain_" + n], EPS, dy, s["thw"], s["clips"], s["dims"], THETA, dx=dy)
    else:
        got["dq"] = vfm.vfm_rope3d(dq, s["thw"], s["clips"], s["dims"], THETA, inverse=True)
        got["dk"] = vfm.vfm_rope3d(dk, s["thw"], s["clips"], s["dims"], THETA, inverse=True)
    return got


def _run_cross(s):
    q, k, v, cq, ck, scale = s["q"], s["k"], s["v"], s["cu_q"], s["cu_k"], s["scale"]
    if not s["case"]["train"]:
        out, lse = vfm.vfm_xattn_fwd(q, k, v, cq, ck, scale, out=s["out"], lse=s["lse"])
        return {"out": out, "lse": lse}
    out, lse = vfm.vfm_xattn_fwd(q, k, v, cq, ck, scale)
    dq, dk, dv = vfm.vfm_xattn_bwd(q, k, v, out, lse, s["dout"], cq, ck, scale, workspace=s["workspace"])
    return {"out": out, "lse": lse, "dq": dq, "dk": dk, "dv": dv}


def _run_temporal(s):
    q, k, v, thw, cu, scale = s["q"], s["k"], s["v"], s["thw"], s["clips"], s["scale"]
    if not s["case"]["train"]:
        return {"out": vfm.vfm_tattn_fwd(q, k, v, thw, cu, scale, out=s["out"])}
    out = vfm.vfm_tattn_fwd(q, k, v, thw, cu, scale)
    dq, dk, dv = vfm.vfm_tattn_bwd(q, k, v, s["dout"], thw, cu, scale)
    return {"out": out, "dq": dq, "dk": dk, "dv": dv}


def _run_fp8(s):
    q, k = _encode(s)
    q8, k8, v8, scales = vfm.vfm_fp8_pack(q, k, s["v"], s["clips"], s["scale"], *s["packed"])
    out, lse = vfm.vfm_attn_fwd_fp8(q8, k8, v8, scales, s["clips"], s["case"]["heads"], s["case"]["head_dim"],
                                    out=s["out"], lse=s["lse"])
    return {"q": q, "k": k, "out": out, "lse": lse}


_PATHS = {"self": _run_self, "cross": _run_cross, "temporal": _run_temporal, "fp8": _run_fp8}


def run(state):
    return _PATHS[state["case"]["path"]](state)


def work(case):
    """Per call: every tensor it takes read once, every tensor it gives written once, and the
    matrix products over the (query, key) pairs of each sequence (4 D forward, 10 D backward)."""
    heads, hd, path, train = case["heads"], case["head_dim"], case["path"], case["train"]
    total = sum(_lengths(case["grids"]))
    lens_q, lens_k = _sequences(case)
    big = 2.0 * total * heads * hd                                  # one query-sized bf16 tensor
    kv = 2.0 * (sum(lens_k) if path == "cross" else total) * heads * hd
    lse = 4.0 * total * heads
    if path == "temporal":
        pairs = sum(t * t * h * w for t, h, w in _grids(case["grids"]))
        bytes_ = 4 * big + (7 * big if train else 0)
    else:
        pairs = sum(a * b for a, b in zip(lens_q, lens_k))
        bytes_ = 2 * big + 2 * kv + lse                             # q, out; k, v
        if train:
            bytes_ += 4 * big + 4 * kv + lse                        # q, out, dout, dq; k, v, dk, dv
        if path != "cross":
            bytes_ += 4 * big                                       # position encoding of q and k
            if train:
                bytes_ += (6 if case["encode"] == "qknorm" else 4) * big
        if path == "fp8":
            bytes_ += 3 * big                                       # packed q, k, v: written once, read once
    return {"bytes": bytes_, "flops": float(4 + (10 if train else 0)) * hd * heads * pairs}


def tolerance(case):
    # Against 64-bit arithmetic on the same bf16 inputs outputs and gradients are off by 2.0e-3 to
    # 4.2e-3 in the 2-norm (the bf16 rounding of results, of P and dS and of what one call hands to
    # the next), single values by at most 0.07 of the root mean square (rows of a gradient that are
    # small by cancellation): two or three times that in the norm, four times in the largest.
    # 8-bit operands: P carries three mantissa bits (2.0e-2 to 2.7e-2 against 64-bit arithmetic on the same codes).
    if case["path"] == "fp8":
        return {"rel": 0.03, "max": 0.5}
    return {"rel": 1e-2, "max": 0.25}
