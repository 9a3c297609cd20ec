"""The calls that users of the library time: single tokens and prefills through the forward pass,
training steps of the block loop (dense, masked, float32), whole layers under activation
recomputation, and the projections by themselves.

A case is a dict of plain values:

  kind      "decode"  lvx_xattn_fwd with a few query rows against all visual keys (serving)
            "prefill" BlockLoop.forward (a prompt's text against the visual keys, in K/V blocks)
            "train"   BlockLoop.forward + BlockLoop.backward (a training step's cross-attention)
            "layer"   RecomputeLayer.forward + .backward (the same from token features, with the
                      projections run again in the backward pass and their gradients)
            "project" lvx_xattn_project + lvx_xattn_project_bwd (K, V of a block of visual tokens
                      and the gradients carried back to the tokens and the weights)
  dtype     "bf16" or "f32";  B, Hq, Hkv, D, Sq, Skv as in the library's interface
  blocks    K/V blocks that the query rows visit in turn
  q_chunk, kv_block, mask   media mask: text rows per chunk, visual tokens per frame, "causal" (a
                      chunk sees the frames up to its own) or "recent" (only its own); 0, 0, "" = dense
  outliers  1 % of the key tokens carry eight times the others' magnitude
  E         embedding width of the token features ("layer", "project")

`listed` holds the shapes that the repository's workloads name, one for each kind of use;
`draw` gives others of the same ranges.
"""
from __future__ import annotations

import math

import torch

from paper_2502_02406_amd import binding as B
from paper_2502_02406_amd import workloads as W
from paper_2502_02406_amd.blockloop import BlockLoop, MediaMask, RecomputeLayer


def _case(kind, Hq, Hkv, D, Sq, Skv, *, dtype="bf16", B=1, blocks=1, q_chunk=0, kv_block=0, mask="",
          outliers=False, E=0):
    return dict(kind=kind, dtype=dtype, B=B, Hq=Hq, Hkv=Hkv, D=D, Sq=Sq, Skv=Skv, blocks=blocks,
                q_chunk=q_chunk, kv_block=kv_block, mask=mask, outliers=outliers, E=E)


def listed():
    return [
        # serving, one generated token: against a single image of 6404 visual tokens (launches and
        # latency), and against a long video of 256 frames (K and V are read once)
        dict(_case("decode", 32, 8, 128, 1, 6404), name="decode_one_image"),
        dict(_case("decode", 32, 8, 128, 1, 262144), name="decode_long_video"),
        # serving, a prompt: the Video-MME text length against ten frames of 6404 tokens, two blocks
        dict(_case("prefill", 32, 8, 128, 5514, 64040, blocks=2), name="prefill_ragged"),
        # training, dense: Llama-3-V-like layer in two blocks of 32768 keys; one worker's share of the
        # text with 729-token frames and head groups of 7; 64-wide heads with 64-token frames
        dict(_case("train", 32, 8, 128, 2048, 65536, blocks=2), name="train_llama"),
        dict(_case("train", 28, 4, 128, 512, 182250, blocks=2), name="train_owl_729"),
        dict(_case("train", 8, 8, 64, 4096, 131072), name="train_flamingo_64"),
        # training under a media mask: text chunks and frames made of whole tiles; frames of 729
        # tokens, which no tile divides; two text tokens per frame, each pair sees its frame only
        dict(_case("train", 16, 16, 128, 1024, 131072, B=2, q_chunk=32, kv_block=1024, mask="causal"),
             name="train_masked_frames"),
        dict(_case("train", 28, 4, 128, 2048, 23328, q_chunk=64, kv_block=729, mask="causal"),
             name="train_masked_729"),
        dict(_case("train", 8, 8, 64, 4096, 131072, q_chunk=2, kv_block=64, mask="recent"),
             name="train_recent_frame"),
        # the exact check in float32: a tiny layer in four blocks
        dict(_case("train", 2, 2, 64, 128, 1024, dtype="f32", blocks=4), name="train_f32_tiny"),
        # a layer from its token features (an 8B language model's width), one block of visual tokens
        dict(_case("layer", 32, 8, 128, 2048, 32768, E=4096), name="layer_wide"),
        # K, V of a block from a narrow visual encoder's features, and their gradients
        dict(_case("project", 0, 8, 64, 0, 131072, E=512), name="project_narrow"),
    ]


# ---- further cases --------------------------------------------------------------------------

_HEADS = ((32, 8, 128), (28, 4, 128), (16, 16, 128), (8, 8, 64), (32, 8, 64), (32, 8, 96))
_MOST_FLOPS = 0.9 * 14.0 * 32 * 2048 * 65536 * 128      # "train_llama", the largest listed case


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    """A size in [lo, hi], even over its logarithm: a power of two, a multiple of 64, or any number."""
    n = _log(rng, lo, hi)
    how = rng.randrange(4)
    if how == 0:
        n = 1 << round(math.log2(n))
    elif how == 1:
        n = (n + 63) // 64 * 64
    return max(lo, min(hi, n))


def draw(rng):
    kind = rng.choice(("decode", "decode", "prefill", "train", "train", "train", "masked", "masked",
                       "f32", "layer", "project"))
    Hq, Hkv, D = rng.choice(_HEADS)
    if kind == "decode":
        Bn = _log(rng, 1, 8)
        most = (1 << 30) // (Bn * Hkv * D * 2)              # at most 1 GiB of keys
        return _case("decode", Hq, Hkv, D, rng.choice((1, 1, 1, _log(rng, 2, 16))),
                     _size(rng, 1024, min(most, 1 << 20)), B=Bn, outliers=rng.random() < 0.25)
    if kind in ("prefill", "train"):
        units = 4.0 if kind == "prefill" else 14.0
        Sq = _size(rng, 64, 8192)
        most = _MOST_FLOPS / (units * Hq * Sq * D)
        blocks = rng.choice((1, 2, 4))
        per = _size(rng, 1024, int(min(most, 262144)) // blocks)
        return _case(kind, Hq, Hkv, D, Sq, per * blocks, blocks=blocks, outliers=rng.random() < 0.25)
    if kind == "masked":
        mask = rng.choice(("causal", "recent"))
        frame = rng.choice((64, 64, 256, 729, 1024, 1601))
        chunk = rng.choice((2, 8, 16, 32, 64, rng.randint(3, 100)))
        frames = _log(rng, 8, min(2048, 131072 // frame))
        Sq = max(64, min(4096, chunk * _log(rng, max(4, frames // 2), 2 * frames) - rng.choice((0, 0, 1))))
        Bn = rng.choice((1, 1, 2)) if Hkv * frame * frames * D <= 1 << 27 else 1
        c = _case("train", Hq, Hkv, D, Sq, frame * frames, B=Bn, q_chunk=chunk, kv_block=frame, mask=mask)
        while work(c)["flops"] > _MOST_FLOPS:
            c["Sq"] //= 2
        return c
    if kind == "f32":
        Hq, Hkv = rng.choice(((2, 2), (4, 2), (8, 8)))
        blocks = rng.choice((1, 4))
        return _case("train", Hq, Hkv, rng.choice((64, 96, 128)), _size(rng, 16, 512),
                     blocks * _size(rng, 64, 4096 // blocks), dtype="f32", blocks=blocks)
    E = rng.choice((512, 1024, 2048, 4096))
    if kind == "layer":
        Sq = _size(rng, 128, 4096)
        blocks = rng.choice((1, 1, 2))
        most = _MOST_FLOPS / (18.0 * Hq * Sq * D + 16.0 * E * Hkv * D)
        return _case("layer", Hq, Hkv, D, Sq, blocks * _size(rng, 1024, int(min(most, 65536)) // blocks),
                     blocks=blocks, E=E)
    most = _MOST_FLOPS / (12.0 * E * Hkv * D)
    return _case("project", 0, Hkv, D, 0, _size(rng, 2048, int(min(most, 131072))), E=E)


# ---- one case -------------------------------------------------------------------------------

def prepare(case, seed):
    c = case
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dt = W.torch_dtype(c["dtype"])
    std = 1.0 if c["dtype"] == "f32" else 0.5

    def normal(*shape, std=std):
        # (drawn in place, a head at a time: no second copy of the tensor in float32)
        out = torch.empty(shape, dtype=dt, device="cuda")
        for part in out.view(-1, *shape[-2:]):
            part.copy_(torch.randn(shape[-2:], generator=g, device="cuda") * std)
        return out

    Bn, Hq, Hkv, D, Sq, Skv, E = (c[n] for n in ("B", "Hq", "Hkv", "D", "Sq", "Skv", "E"))
    if c["kind"] == "project":
        return {"case": c, "y": normal(1, Skv, E, std=1.0), "wkv": normal(2 * Hkv * D, E, std=0.5 / E ** 0.5),
                "grads": [normal(1, Hkv, Skv, D, std=0.05) for _ in range(2)],
                "heads": [torch.empty((1, Hkv, Skv, D), dtype=dt, device="cuda") for _ in range(2)],
                "dy": torch.empty((1, Skv, E), dtype=dt, device="cuda"),
                "dw": torch.zeros((2 * Hkv * D, E), dtype=torch.float32, device="cuda")}
    if c["kind"] == "layer":
        return {"case": c, "x": normal(Bn, Sq, E, std=1.0), "y": normal(Bn, Skv, E, std=1.0),
                "wq": normal(Hq * D, E, std=0.5 / E ** 0.5), "wkv": normal(2 * Hkv * D, E, std=0.5 / E ** 0.5),
                "do": normal(Bn, Hq, Sq, D),
                "layer": RecomputeLayer(Bn, Sq, Skv, E, Hq, Hkv, D, dt, c["blocks"])}
    s = {"case": c, "q": normal(Bn, Hq, Sq, D), "k": normal(Bn, Hkv, Skv, D), "v": normal(Bn, Hkv, Skv, D)}
    if c["outliers"]:
        tok = torch.randperm(Skv, generator=g, device="cuda")[:max(1, Skv // 100)]
        s["k"][:, :, tok] *= 8.0
    if c["kind"] == "decode":
        s["p"] = B.make_problem(s["q"], s["k"])
        n = B.lvx_xattn_workspace_bytes(s["p"], B.dtype_code(dt), B.LVX_WS_FWD)
        s["ws"] = torch.empty(n, dtype=torch.uint8, device="cuda")
        s["o"] = torch.empty_like(s["q"])
        s["lse"] = torch.empty((Bn, Hq, Sq), dtype=torch.float32, device="cuda")
        return s
    mask = None
    if c["mask"]:
        allow = torch.from_numpy(W.media_mask(_workload(c))).cuda()
        mask = MediaMask(allow, c["q_chunk"], c["kv_block"])
    s["loop"] = BlockLoop((Bn, Hq, Sq, D), (Bn, Hkv, Skv, D), dt, c["blocks"], mask)
    if c["kind"] == "train":
        s["do"] = normal(Bn, Hq, Sq, D)
        s["dk"], s["dv"] = torch.empty_like(s["k"]), torch.empty_like(s["v"])
    return s


def run(state):
    s = state
    kind = s["case"]["kind"]
    if kind == "decode":
        B.lvx_xattn_fwd(s["p"], s["q"], s["k"], s["v"], None, s["o"], s["lse"], s["ws"])
        return s["o"], s["lse"]
    if kind == "prefill":
        return s["loop"].forward(s["q"], s["k"], s["v"])
    if kind == "train":
        o, lse = s["loop"].forward(s["q"], s["k"], s["v"])
        dq = s["loop"].backward(s["q"], s["k"], s["v"], o, lse, s["do"], s["dk"], s["dv"])
        return o, lse, dq, s["dk"], s["dv"]
    if kind == "layer":
        o, lse = s["layer"].forward(s["x"], s["y"], s["wq"], s["wkv"])
        return (o, lse) + s["layer"].backward(s["x"], s["y"], s["wq"], s["wkv"], o, lse, s["do"])
    s["dw"].zero_()
    B.lvx_xattn_project(s["y"], s["wkv"], s["heads"])
    B.lvx_xattn_project_bwd(s["y"], s["wkv"], s["grads"], dx=s["dy"], dw=s["dw"])
    return s["heads"][0], s["heads"][1], s["dy"], s["dw"]


def _workload(c):
    return W.Workload("case", B=c["B"], Hq=c["Hq"], Hkv=c["Hkv"], D=c["D"], Sq=c["Sq"], Skv=c["Skv"],
                      dtype=c["dtype"], std=1.0, q_chunk=c["q_chunk"], kv_block=c["kv_block"],
                      mask_kind=c["mask"] or "causal")


def work(case):
    """Each input read once and each output written once by the forward and by the backward pass;
    the matrix products that the definition asks for (4 units of query x key x head x width
    forward, 10 backward; visible pairs only)."""
    c = case
    e = 4 if c["dtype"] == "f32" else 2
    kv = c["B"] * c["Hkv"] * c["Skv"] * c["D"]
    q = c["B"] * c["Hq"] * c["Sq"] * c["D"]
    rows = c["B"] * c["Hq"] * c["Sq"]
    if c["kind"] == "project":
        M, N, E = c["Skv"], 2 * c["Hkv"] * c["D"], c["E"]
        fwd = (M * E + N * E + M * N) * e
        bwd = (M * N + N * E + M * E) * e + M * E * e + N * E * 4
        return {"bytes": fwd + bwd, "flops": 6.0 * M * N * E}
    units = c["B"] * c["Hq"] * c["D"] * float(c["Sq"]) * c["Skv"]
    seen = kv
    if c["mask"]:
        w = _workload(c)
        units = c["B"] * c["Hq"] * c["D"] * w.visible_pairs()
        on = W.media_mask(w).any(axis=0)
        seen = c["B"] * c["Hkv"] * c["D"] * min(c["Skv"], int(on.sum()) * c["kv_block"])
    fwd = (2 * q + 2 * seen) * e + rows * 4
    if c["kind"] in ("decode", "prefill"):
        return {"bytes": fwd, "flops": 4.0 * units}
    bwd = (3 * q + 2 * seen) * e + rows * 4 + (q + 2 * kv) * e      # Q, O, dO, K, V, L; dQ, dK, dV
    if c["kind"] == "train":
        return {"bytes": fwd + bwd, "flops": 14.0 * units}
    # the layer: features and weights instead of Q, K, V; projections forward, again, and their gradients
    E, tx, ty = c["E"], c["B"] * c["Sq"], c["B"] * c["Skv"]
    nq, nkv = c["Hq"] * c["D"], 2 * c["Hkv"] * c["D"]
    nbytes = (3 * (tx + ty) * E + 2 * (nq + nkv) * E + 3 * q) * e + (nq + nkv) * E * 4 + 2 * rows * 4
    return {"bytes": nbytes, "flops": 14.0 * units + 8.0 * E * (tx * nq + ty * nkv)}


def tolerance(case):
    """Four times the distance, measured on shapes of these ranges, from the same path evaluated in
    float64: float32 1.3e-6, a little more over longer sums; bfloat16 2.4e-3 (its rounding of the
    results and of the probabilities), 4.7e-3 for gradients where outlying keys make large scores,
    with single elements off by 0.25 of the root mean square there."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    if case["outliers"]:
        return {"rel": 2e-2, "max": 0.9}
    return {"rel": 1e-2}
