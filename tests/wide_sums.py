"""Blocks whose integer sums reach a given size: rows of weights of one sign and a given sum of magnitudes, LayerNorms and an attention that drive
every input code to the end farther from its zero point."""
import numpy as np

from paper_2507_19131_amd import synth

LAYERS = ("qkv", "proj", "fc1")
WIDEST = 16448                                            # * 255 = 2^22 - 64: the widest rows whose 8-bit sums stay below 2^22


def _row(K, width, sign):
    """K codes of one sign whose magnitudes add up to `width`, or as near as int8 holds."""
    row = np.full(K, width // K)
    row[:width % K] += 1
    return np.minimum(row, 127 if sign > 0 else 128) * sign


def make_inputs(spec, widths, sign=1, seed=58):
    """widths: of the rows of (w_qkv, w_proj, w_fc1); the sums of the high branch reach 255 times that at 8 bits, of either sign (v: of sign `sign`,
    which the attention hands on to the projection).  The dequantized values stay well inside their quantizers."""
    spans = {"a_qkv_in": 3.0, "a_proj_in": 0.4, "a_fc1_in": 3.0}          # of the input codes, in real units
    inp = synth.make_block_inputs(spec, seed, ranges={q: (0.0, v) if sign > 0 else (-v, 0.0) for q, v in spans.items()})
    for br in inp.branches:
        for n in ("ln1", "ln2"):
            getattr(br, n + "_gamma")[:] = 1e-3
            getattr(br, n + "_beta")[:] = 10.0 * sign
    C = spec.C
    for layer, width, span in zip(LAYERS, widths, spans.values()):
        w = getattr(inp.shared, "w_" + layer)
        pos, neg = _row(C, width, 1), _row(C, width, -1)
        w[0::2], w[1::2] = pos, neg
        if layer == "qkv":
            w[2 * C:] = pos
        getattr(inp.shared, "s_" + layer)[:] = 0.6 / (span * width)
    return inp
