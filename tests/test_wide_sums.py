"""The blocks of wide_sums.py do what the GPU tests rely on, and taking a sum beyond 2^22 for its own bits shows in them.  CPU only."""
import numpy as np
import pytest

import oracle_api as O
import wide_sums
from paper_2507_19131_amd import synth

BOUND = 1 << 22


def as_its_own_bits(acc):
    """1.5 * 2^23 + sum as the bits of a binary32, less 1.5 * 2^23."""
    return (acc.astype(np.int64) + 0x4B400000).astype(np.uint32).view(np.float32).astype(np.float64) - 1.5 * 2**23


@pytest.mark.parametrize("C,width,sign", [(128, 16384, 1), (192, 16448, 1), (192, 16448, -1), (192, 16449, 1), (192, 16449, -1), (192, 20480, 1),
                                          (192, 20480, -1), (384, 16448, 1), (384, 20480, 1)])
def test_every_layer_reaches_its_sum(C, width, sign):
    spec = synth.BlockSpec(1, 14, 14, C, C // 32, shift=3)
    inp = wide_sums.make_inputs(spec, (width, width, width), sign)
    x = synth.make_feature_map(spec, 58, blobs=True)
    perm = O.select_windows(O.score_windows(inp, x), 2)
    _, taps = O.block_forward(inp, x, perm, 2, want_taps=("acc_qkv", "acc_proj", "acc_fc1"))
    for name, acc in taps.items():
        acc = acc[:2]                                       # the high branch
        reached = (int(acc.min()), int(acc.max()))
        positive, negative = (min(width, 127 * C), width) if sign > 0 else (width, min(width, 127 * C))
        assert reached == (-255 * negative, 255 * positive), (name, reached)
        wrong = np.abs(as_its_own_bits(acc) - acc)
        if width <= wide_sums.WIDEST:
            assert max(-reached[0], reached[1]) < BOUND and wrong.max() == 0, name
        else:
            assert max(-reached[0], reached[1]) >= BOUND and wrong.max() > 0, name
        if width > 20000:                                   # by 10 % of values that span several codes
            assert (wrong > 0.08 * np.abs(acc)).any(), name
