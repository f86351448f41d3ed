"""The performance cases of the Two-Branch Swin Block library: what its users run, through the public entry points.

A case is one of
  block     one block on one map, scored and selected inside the call (mixaq_block_forward, perm = NULL)
  stage     a run of blocks on one map with one score and one selection (mixaq_stage_forward)
  embed     the patch embedding, image -> stage 1 (mixaq_downsample_forward, kind 0)
  merge     a patch merging between two stages (mixaq_downsample_forward, kind 1)
  backbone  embedding, four stages and the mergings between them as one chain

Sizes are those of the benchmark's workloads (Swin-T at 800x1344, Swin-B-shaped maps of 1024x1024 images) and the
range around them; weights, quantizers and maps are drawn from the seed on the GPU with the distributions of
paper_2507_19131_amd/synth.py.  Outputs are the maps, the scores and the selection lists, whole.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2507_19131_amd import binding as M
from paper_2507_19131_amd import synth

# quantizer settings in use: (high activation bits, low activation bits, weight bits)
PRECISIONS = ((8, 4, 8), (8, 4, 4), (4, 2, 4))
# clip ranges of maps with outlier channels (the other ranges are synth.DEFAULT_RANGES)
OUTLIER_RANGES = {"a_qkv_in": (-12.0, 13.5), "a_fc1_in": (-11.0, 10.0)}
MAX_GOP = 262.0            # the largest listed stage
WIDTHS = (96, 128, 192, 256, 384, 512, 768, 1024)


def _stage(name, kind, B, H, W, C, blocks, keep, prune=0.0, bits=(8, 4, 8), score_mode=0, own_bias=False, outliers=False):
    case = dict(kind=kind, B=B, H=H, W=W, C=C, blocks=blocks, keep=keep, prune=prune, high=bits[0], low=bits[1], weight=bits[2],
                score_mode=score_mode, own_bias=own_bias, outliers=outliers)
    return dict(case, name=name) if name else case


def listed():
    return [
        # the smallest call: one block on a classification-size map, where launches and latency count
        _stage("block 56x56x96", "block", 1, 56, 56, 96, 1, 0.5),
        # the benchmark's headline: the stage-1 pair of a detection backbone on one image
        _stage("stage 200x336x96", "stage", 1, 200, 336, 96, 2, 0.5),
        # the same stage on a batch, the score taken behind a LayerNorm: throughput once the chip is full
        _stage("stage 8x200x336x96", "stage", 8, 200, 336, 96, 2, 0.5, score_mode=1),
        # stage 2 of the same backbone at the 4-bit setting with 2-bit low windows (QAT)
        _stage("stage 100x168x192 W4", "stage", 1, 100, 168, 192, 2, 0.5, bits=(4, 2, 4)),
        # ragged maps, a third image, pruned windows, biases of their own per branch (PTQ, W4 A8/A4)
        _stage("stage 3x61x93x192 pruned", "stage", 3, 61, 93, 192, 2, 0.4, prune=0.2, bits=(8, 4, 4), own_bias=True),
        # the deep stage 3: six blocks on a small batch of small maps
        _stage("stage 2x50x84x384", "stage", 2, 50, 84, 384, 6, 0.5),
        # stage 4: the widest layers on the fewest windows, the path of separate kernels
        _stage("stage 25x42x768 W4", "stage", 1, 25, 42, 768, 2, 0.5, bits=(4, 2, 4)),
        # the wider backbone's first two stages on a batch, with outlier channels
        _stage("stage 4x256x256x128", "stage", 4, 256, 256, 128, 2, 0.4, outliers=True),
        _stage("stage 4x128x128x256", "stage", 4, 128, 128, 256, 2, 0.4, outliers=True),
        # the layers between stages, each on its own
        dict(name="embed 800x1344", kind="embed", B=1, H=800, W=1344, C=3, N=96, high=8, weight=8),
        dict(name="merge 4x256x256x128", kind="merge", B=4, H=256, W=256, C=128, N=256, high=8, weight=8),
        # one image through the whole backbone, as a detector runs it
        dict(name="backbone 800x1344 W4", kind="backbone", B=1, H=800, W=1344, C=96, keep=0.5, high=4, low=2, weight=4),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(("block", "stage", "stage", "stage", "stage", "stage", "stage", "embed", "merge", "backbone"))
    bits = rng.choice(PRECISIONS)
    if kind in ("block", "stage"):
        C = rng.choice(WIDTHS)
        blocks = 1 if kind == "block" else rng.choice((2, 2, 2, 6))
        per_window = 2e-9 * _macs_per_window(C) * blocks
        windows = min(max(_log_uniform(rng, 0.75, MAX_GOP) / per_window, 4.0), MAX_GOP / per_window)
        B = rng.choice((1, 1, 1, 2, 3, 4, 8))
        while B > 1 and windows / B < 4:
            B -= 1
        per_image = min(windows / B, 3600.0)
        aspect = _log_uniform(rng, 0.6, 1.7)
        # round the windows down, then take an unpadded size inside the last row and column of windows
        rows = max(2, int(math.sqrt(per_image / aspect)))
        cols = max(2, int(per_image / rows))
        H, W = 7 * rows - rng.randrange(7), 7 * cols - rng.randrange(7)
        return _stage(None, kind, B, H, W, C, blocks, rng.choice((0.25, 0.4, 0.5, 0.75)), prune=rng.choice((0.0, 0.0, 0.2)), bits=bits,
                      score_mode=rng.choice((0, 0, 1)), own_bias=rng.random() < 0.5, outliers=rng.random() < 0.25)
    if kind == "embed":
        side = _log_uniform(rng, 224, 1344)
        return dict(kind="embed", B=rng.choice((1, 2, 4)), H=int(side), W=int(side * _log_uniform(rng, 0.7, 1.4)), C=3,
                    N=rng.choice((96, 128)), high=bits[0], weight=bits[2])
    if kind == "merge":
        C = rng.choice((96, 128, 192, 256, 384, 512))
        side = _log_uniform(rng, 32, 256) * 128 / C
        H, W = max(14, int(side)), max(14, int(side * _log_uniform(rng, 0.7, 1.4)))
        return dict(kind="merge", B=rng.choice((1, 2, 4)), H=H, W=W, C=C, N=2 * C, high=bits[0], weight=bits[2])
    pixels, B = _log_uniform(rng, 1.6e5, 1.05e6), rng.choice((1, 1, 2))     # of the whole batch: at most about the listed image
    aspect = _log_uniform(rng, 0.7, 1.4)
    H, W = int(math.sqrt(pixels / B / aspect)), int(math.sqrt(pixels / B * aspect))
    return dict(kind="backbone", B=B, H=max(256, H), W=max(256, W), C=96, keep=rng.choice((0.25, 0.5, 0.75)), high=bits[0], low=bits[1],
                weight=bits[2])


# ---------------------------------------------------------------- sizes
def _macs_per_window(C):
    return 588 * C * C + 4802 * C


def _spec(case, **other):
    g = dict(case, **other)
    return synth.BlockSpec(g["B"], g["H"], g["W"], g["C"], g["C"] // 32, act_bits_high=g["high"], act_bits_low=g["low"],
                           weight_bits=g["weight"], score_mode=g.get("score_mode", 0))


def _down_spec(kind, case, **other):
    g = dict(case, **other)
    return synth.DownSpec(kind, g["B"], g["H"], g["W"], g["C"], g["N"], act_bits=g["high"], weight_bits=g["weight"])


def _chain(case):
    """(embedding, [(stage spec, blocks), ...], [mergings]) of a backbone case."""
    embed = _down_spec(0, case, C=3, N=case["C"])
    H, W, C, stages, merges = embed.Ho, embed.Wo, case["C"], [], []
    for i, blocks in enumerate((2, 2, 6, 2)):
        if i:
            merges.append(_down_spec(1, case, H=H, W=W, C=C, N=2 * C))
            H, W, C = merges[-1].Ho, merges[-1].Wo, 2 * C
        stages.append((_spec(case, H=H, W=W, C=C), blocks))
    return embed, stages, merges


def _stage_work(spec, blocks, computed):
    weights = blocks * 12 * spec.C * spec.C
    return (spec.B * spec.H * spec.W * spec.C * 4, weights, 2.0 * _macs_per_window(spec.C) * spec.B * computed * blocks)


def _down_work(d):
    tokens = d.B * d.Ho * d.Wo
    return (d.B * d.H * d.W * d.C_in * 4, d.N * d.K, tokens * d.N * 4, 2.0 * tokens * d.K * d.N)


def work(case):
    """Bytes: the input map or image, the weights (int8) and every map that comes back, once each."""
    if case["kind"] in ("embed", "merge"):
        read, weights, written, ops = _down_work(_down_spec(0 if case["kind"] == "embed" else 1, case))
        return {"bytes": read + weights + written, "flops": ops}
    if case["kind"] == "backbone":
        embed, stages, merges = _chain(case)
        bytes_, ops = embed.B * embed.H * embed.W * 3 * 4, 0.0
        for d in [embed] + merges:
            bytes_ += _down_work(d)[1]
            ops += _down_work(d)[3]
        for spec, blocks in stages:
            out, weights, o = _stage_work(spec, blocks, spec.nW)
            bytes_ += out + weights
            ops += o
        return {"bytes": bytes_, "flops": ops}
    spec = _spec(case)
    k_high, k_low = _counts(case, spec)
    out, weights, ops = _stage_work(spec, case["blocks"], k_high + k_low)
    return {"bytes": 2 * out + weights, "flops": ops}


def tolerance(case):
    """Codes, integer sums and selection lists are defined bit for bit; binary64 reductions that feed a code may be taken
    in another order, which moves at most the last bit of a score and, once in about 1e9 reductions, a binary32 value."""
    return {"rel": 1e-6, "max": 1e-3, "differ": 0.0}


# ---------------------------------------------------------------- inputs
def _normal(gen, *shape):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)


def _weights(gen, n_out, n_in, bits, std=0.02):
    """Symmetric per-output-channel codes in int8 containers and their scales."""
    qmax = (1 << (bits - 1)) - 1
    w = _normal(gen, n_out, n_in) * std
    s = (w.abs().amax(dim=1) / qmax).clamp_min(1e-8)
    return (w / s[:, None]).round().clamp(-qmax, qmax).to(torch.int8), s


def _layernorm(gen, n):
    return (1.0 + 0.25 * _normal(gen, n)).clamp(0.25, 2.0), 0.1 * _normal(gen, n)


def _block_inputs(gen, spec, own_bias, outliers):
    C, F = spec.C, spec.C * spec.mlp_ratio
    sh = SimpleNamespace()
    for name, n_out, n_in in (("qkv", 3 * C, C), ("proj", C, C), ("fc1", F, C), ("fc2", C, F)):
        w, s = _weights(gen, n_out, n_in, spec.weight_bits)
        setattr(sh, "w_" + name, w)
        setattr(sh, "s_" + name, s)
    table = (_normal(gen, spec.heads, (2 * spec.window - 1) ** 2) * 0.5).cpu().numpy()
    sh.rel_pos_bias = torch.from_numpy(np.ascontiguousarray(synth.expand_rel_pos_bias(table, spec.heads, spec.window))).cuda()
    sh.score_gamma, sh.score_beta = _layernorm(gen, C)
    ranges = dict(synth.DEFAULT_RANGES, **(OUTLIER_RANGES if outliers else {}))
    bias = [0.02 * _normal(gen, n) for n in (3 * C, C, F, C)]
    branches = []
    for i, bits in enumerate((spec.act_bits_high, spec.act_bits_low)):
        br = SimpleNamespace(q={})
        br.ln1_gamma, br.ln1_beta = _layernorm(gen, C)
        br.ln2_gamma, br.ln2_beta = _layernorm(gen, C)
        if i == 1 and own_bias:
            bias = [0.02 * _normal(gen, n) for n in (3 * C, C, F, C)]
        br.b_qkv, br.b_proj, br.b_fc1, br.b_fc2 = bias
        for name in synth.QNAMES:
            lo, hi = ranges[name]
            if i == 1:
                lo, hi = lo * 0.9375, hi * 0.9375
            br.q[name] = synth.qparam_for_range(lo, hi, bits, symmetric=name in ("a_q", "a_k", "a_v"))
        branches.append(br)
    return sh, branches


def _blobs(gen, x, gain, shift_by, count=14):
    """Raises elliptical regions of a [B,H,W,C] map: about a third of it, each with a channel signature of its own."""
    B, H, W, C = x.shape
    rr = torch.arange(H, device="cuda", dtype=torch.float32)[:, None]
    cc = torch.arange(W, device="cuda", dtype=torch.float32)[None, :]
    for b in range(B):
        u = torch.rand((count, 4), generator=gen, device="cuda").cpu().numpy()
        sig = _normal(gen, count, C)
        for k in range(count):
            ay, ax = (0.04 + 0.08 * u[k, 2]) * H + 2, (0.04 + 0.08 * u[k, 3]) * W + 2
            inside = (((rr - float(u[k, 0]) * H) / float(ay)) ** 2 + ((cc - float(u[k, 1]) * W) / float(ax)) ** 2 <= 1.0)[..., None]
            x[b] = torch.where(inside, gain * x[b] + shift_by * sig[k], x[b])
    return x


def _feature_map(gen, spec, outliers):
    x = _normal(gen, spec.B, spec.H, spec.W, spec.C)
    if outliers:
        ch = torch.randperm(spec.C, generator=gen, device="cuda")[:max(1, round(0.03 * spec.C))]
        x[..., ch] *= torch.exp(math.log(8.0) + math.log(4.0) * torch.rand(ch.numel(), generator=gen, device="cuda"))
        return x
    return _blobs(gen, x, 4.0, 3.0)


def _image(gen, B, H, W):
    n = _normal(gen, B * 3, 1, H + 15, W + 15)
    img = 16.0 * torch.nn.functional.avg_pool2d(n, 16, stride=1)
    return _blobs(gen, img.view(B, 3, H, W).permute(0, 2, 3, 1).contiguous(), 2.0, 1.0, count=12)


# ---------------------------------------------------------------- states
class _Blocks:
    """Block handles, destroyed with the state."""

    def __init__(self, gen, spec, blocks, own_bias, outliers):
        self.handles = []
        for i in range(blocks):                         # regular and shifted blocks alternate
            shared, branches = _block_inputs(gen, spec, own_bias, outliers)
            self.handles.append(M.mixaq_block_create(M.make_desc(spec, 3 if i % 2 else 0), shared, branches))
        self.workspace = M.alloc_workspace(self.handles[0])

    def __del__(self):
        for h in self.handles:
            M.mixaq_block_destroy(h)


class _Layer:
    """A layer between stages, destroyed with the state."""

    def __init__(self, gen, d):
        n_ln = d.N if d.kind == 0 else d.K
        w, s = _weights(gen, d.N, d.K, d.weight_bits, 0.2 if d.kind == 0 else 0.02)
        gamma, beta = _layernorm(gen, n_ln)
        p = SimpleNamespace(w=w, s_w=s, bias=0.02 * _normal(gen, d.N) if d.kind == 0 else None, ln_gamma=gamma, ln_beta=beta,
                            a_in=synth.qparam_for_range(-4.0, 4.5, d.act_bits))
        self.handle = M.mixaq_downsample_create(M.make_downsample_desc(d), p)
        self.y = torch.empty((d.B, d.Ho, d.Wo, d.N), device="cuda")

    def __del__(self):
        if hasattr(self, "handle"):
            M.mixaq_downsample_destroy(self.handle)


def _counts(case, spec):
    """(k_high, k_low) per image from the keep and prune ratios."""
    k_high = int(math.floor(case["keep"] * spec.nW + 0.5))
    pruned = int(math.floor(case.get("prune", 0.0) * spec.nW + 0.5))
    return k_high, max(0, spec.nW - k_high - pruned)


def _stage_state(gen, spec, blocks, k_high, k_low, own_bias=False, outliers=False):
    pairs = (blocks + 1) // 2
    return SimpleNamespace(blocks=_Blocks(gen, spec, blocks, own_bias, outliers), k_high=[k_high] * pairs,
                           k_low=[k_low] * pairs if k_high + k_low < spec.nW else None,
                           y=torch.empty((spec.B, spec.H, spec.W, spec.C), device="cuda"),
                           tmp=torch.empty((spec.B, spec.H, spec.W, spec.C), device="cuda"),
                           scores=torch.empty((spec.B, spec.nW), dtype=torch.float64, device="cuda"),
                           perm=torch.empty((spec.B, spec.nW), dtype=torch.int32, device="cuda"))


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    kind = case["kind"]
    if kind in ("embed", "merge"):
        d = _down_spec(0 if kind == "embed" else 1, case)
        x = _image(gen, d.B, d.H, d.W) if kind == "embed" else _blobs(gen, _normal(gen, d.B, d.H, d.W, d.C_in), 4.0, 3.0)
        return SimpleNamespace(kind=kind, x=x, layer=_Layer(gen, d))
    if kind == "backbone":
        embed, stages, merges = _chain(case)
        return SimpleNamespace(kind=kind, x=_image(gen, case["B"], case["H"], case["W"]), layers=[_Layer(gen, d) for d in [embed] + merges],
                               stages=[_stage_state(gen, s, n, *_counts(case, s)) for s, n in stages])
    spec = _spec(case)
    k_high, k_low = _counts(case, spec)
    state = _stage_state(gen, spec, case["blocks"], k_high, k_low, case["own_bias"], case["outliers"])
    state.kind, state.x = kind, _feature_map(gen, spec, case["outliers"])
    state.prunes = k_high + k_low < spec.nW
    return state


def _run_stage(s, x):
    M.mixaq_stage_forward(s.blocks.handles, x, s.k_high, s.k_low, s.y, s.tmp, s.scores, s.perm, s.blocks.workspace)
    return {"y": s.y, "scores": s.scores, "perm": s.perm}


def run(state):
    if state.kind in ("embed", "merge"):
        return M.mixaq_downsample_forward(state.layer.handle, state.x, state.layer.y)
    if state.kind == "backbone":
        x, maps = state.x, []
        for layer, stage in zip(state.layers, state.stages):
            M.mixaq_downsample_forward(layer.handle, x, layer.y)
            maps.append(_run_stage(stage, layer.y))
            x = stage.y
        return maps
    if state.kind == "block":
        h = state.blocks.handles[0]
        if state.prunes:
            return M.mixaq_block_forward_pruned(h, state.x, None, state.k_high[0], state.k_low[0], state.y, state.blocks.workspace)
        return M.mixaq_block_forward(h, state.x, None, state.k_high[0], state.y, state.blocks.workspace)
    return _run_stage(state, state.x)
