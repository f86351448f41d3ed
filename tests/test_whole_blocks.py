"""Blocks of few windows that one kernel takes whole (csrc/block_plan.h) against the separate kernels, bit for bit, and the rule itself."""
import pytest
import torch

from paper_2507_19131_amd import binding as M
from paper_2507_19131_amd import synth
import gpu_harness as gh
import stage_plan
from test_kernel_resources import kernels, workgroups_per_cu      # noqa: F401 (a fixture)

whole_block = stage_plan.lib.whole_block


@pytest.mark.parametrize("C", [96, 128, 192, 256, 384, 512, 768, 1024])
def test_only_the_widths_that_have_the_kernel_and_only_what_fits_the_chip_at_once(C):
    per_cu = {96: 2, 128: 2, 192: 1}.get(C, 0)
    for windows in range(0, 1100):
        for computed in {0, windows // 2, windows * 4 // 5, windows}:
            if whole_block(C, windows, computed, 0):
                assert 0 < per_cu and computed <= 256 * per_cu and windows <= 512
            if whole_block(C, windows, computed, 1):                 # which of them are pruned shows in the kernel: all take a place
                assert windows <= 256 or computed > 256
                assert windows <= 256 * per_cu and whole_block(C, windows, computed, 0)


@pytest.mark.parametrize("scored", [0, 1])
@pytest.mark.parametrize("NH,per_cu", [(3, 2), (4, 2), (6, 1)])
def test_workgroups_of_a_cu(kernels, NH, scored, per_cu):             # noqa: F811
    """What the rule counts on, by registers and by whole units of LDS."""
    assert workgroups_per_cu(kernels["_ZN5mixaq12block_kernelILi%dELb%dEEEvNS_4GeomENS_7WinArgsENS_7TokArgsE" % (NH, scored)]) == per_cu


# What tells the forms apart: the window kernel hands codes and pixels to the token kernel through the workspace, the whole block nothing.
UNTOUCHED = 0x5A


def _untouched(ws):
    return bool((ws == UNTOUCHED).all())


# B, rows and columns of windows, pruned share: the smallest, ragged and both ends of each range
MAPS = {96: ((1, 1, 1, 0.0), (3, 3, 5, 0.4), (1, 16, 16, 0.0), (2, 10, 14, 0.2), (1, 16, 22, 0.0), (2, 16, 16, 0.0)),
        128: ((1, 12, 12, 0.0), (1, 16, 16, 0.0), (1, 16, 16, 0.2), (2, 10, 14, 0.2), (1, 20, 20, 0.0), (2, 16, 16, 0.0)),
        192: ((1, 12, 12, 0.0), (2, 8, 16, 0.0), (1, 16, 16, 0.2), (2, 10, 14, 0.2), (1, 16, 20, 0.2))}


def _counts(n, pruned):
    k_high = n // 3 if n > 1 else 1
    return k_high, max(0, min(n - n // 3 - int(pruned * n), n - k_high))


def _compare(spec, shifts, k_high, k_low, expect, ranges=None):
    """Given a list, given scores and scored inside the call: the bits of the separate kernels, in the form that is expected."""
    inp = synth.make_block_inputs(spec, 31 + spec.C, ranges=ranges)
    x = torch.from_numpy(synth.make_feature_map(spec, 31 + spec.nW, blobs=True)).cuda()
    for shift in shifts:
        with gh.GpuBlock(inp, shift) as gb, gh.GpuBlock(inp, shift, fused=0) as parts:
            scores, perm = gb.score_select(x, k_high)
            y = parts.forward_pruned(x, perm, k_high, k_low)
            assert not torch.isnan(y).any()
            gb.ws.fill_(UNTOUCHED)
            assert torch.equal(gb.forward_pruned(x, perm, k_high, k_low), y)
            assert _untouched(gb.ws) == expect(0)
            y2, p2 = torch.full_like(x, float("nan")), torch.full_like(perm, -1)
            gb.ws.fill_(UNTOUCHED)
            M.mixaq_block_forward_scored(gb.blk, x, scores, k_high, k_low, y2, gb.ws, perm_out=p2)
            assert torch.equal(y2, y) and torch.equal(p2, perm)
            assert _untouched(gb.ws) == expect(1)
            assert torch.equal(gb.forward_pruned(x, None, k_high, k_low), y)


@pytest.mark.gpu
@pytest.mark.parametrize("bits", [(8, 4, 8), (8, 2, 4), (4, 8, 8)])
@pytest.mark.parametrize("C,B,rows,cols,pruned", [(C, *m) for C, maps in MAPS.items() for m in maps])
def test_whole_blocks_have_the_bits_of_the_separate_kernels(C, B, rows, cols, pruned, bits):
    """Both shifts, given list and scores, both branches' widths packed (2 and 4 bits) and not: whole maps of both forms, and the lists."""
    spec = synth.BlockSpec(B, 7 * rows - 3, 7 * cols - 5, C, C // 32, act_bits_high=bits[0], act_bits_low=bits[1], weight_bits=bits[2])
    n = spec.nW
    k_high, k_low = _counts(n, pruned)
    form = lambda scored: bool(whole_block(C, B * n, B * (k_high + k_low), scored))
    assert n == rows * cols and form(0)
    print("whole block", C, B, rows, cols, pruned, bits, flush=True)
    _compare(spec, (0, 3) if min(rows, cols) > 1 else (0,), k_high, k_low, form)      # a shift needs two windows either way


# the nearest maps outside of the rule, and a block inside of it whose GELU has no table of steps
@pytest.mark.gpu
@pytest.mark.parametrize("C,B,rows,cols,pruned,ranges", [
    (96, 1, 1, 257, 0.0, None), (96, 1, 13, 27, 0.0, None), (96, 1, 19, 27, 0.0, None), (128, 1, 11, 13, 0.0, None), (128, 1, 1, 257, 0.0, None),
    (128, 3, 7, 19, 0.0, None), (128, 1, 19, 27, 0.0, None), (192, 1, 11, 13, 0.0, None), (192, 1, 1, 257, 0.0, None), (192, 3, 7, 18, 0.1, None),
    (96, 1, 4, 5, 0.0, {"a_fc2_in": (-0.07, 0.35)}), (128, 1, 16, 16, 0.2, {"a_fc2_in": (-0.07, 0.35)}), (192, 2, 8, 16, 0.0, {"a_fc2_in": (-0.07, 0.35)})])
def test_blocks_outside_of_the_rule_are_two_kernels(C, B, rows, cols, pruned, ranges):
    spec = synth.BlockSpec(B, 7 * rows, 7 * cols - 2, C, C // 32)
    k_high, k_low = _counts(spec.nW, pruned)
    assert spec.nW == rows * cols
    assert bool(ranges) == bool(whole_block(C, B * spec.nW, B * (k_high + k_low), 0))
    print("two kernels", C, B, rows, cols, pruned, ranges, flush=True)
    _compare(spec, (3,) if rows > 1 else (0,), k_high, k_low, lambda scored: False, ranges)


# B, rows and columns of windows, (high, low) of each pair, blocks whose GELU has no table of steps, whether the stage forks
STAGES = [
    (96, 2, 8, 12, [(48, 48)] * 3, (), False), (128, 2, 16, 16, [(128, 128)] * 3, (), False), (192, 2, 9, 9, [(40, 41)] * 3, (), False),
    (192, 1, 16, 16, [(100, 156), (50, 40), (128, 128)], (), False),          # the second pair computes too few windows for one kernel
    (192, 2, 8, 16, [(64, 64), (30, 30), (64, 64)], (), True),                # the same on a batch
    (96, 1, 16, 16, [(128, 128)] * 2, (1,), False), (192, 2, 8, 16, [(64, 64)] * 3, (4,), True),
    (192, 2, 10, 16, [(80, 48)] * 3, (), False),                              # the first block, which ranks the windows, is two kernels
    (96, 2, 11, 16, [(88, 88)] * 5, (), True)]                                # near two windows a CU a long stage forks


@pytest.mark.gpu
@pytest.mark.parametrize("C,B,rows,cols,counts,cubic,forks", STAGES)
def test_stages_of_whole_blocks(C, B, rows, cols, counts, cubic, forks):
    """Stages whose blocks are one kernel each, or some of them: map, scores and list as block by block through the separate kernels."""
    spec = synth.BlockSpec(B, 7 * rows, 7 * cols - 2, C, C // 32)
    n = 2 * len(counts)
    k_high, k_low = [h for h, _ in counts], [l for _, l in counts]
    windows, L = B * spec.nW, stage_plan.lib
    if cubic:
        assert forks == bool(L.splits(B, spec.nW) and L.pays(B, spec.nW, C, n))
    else:
        assert forks == stage_plan.forks(spec, n, k_high, k_low)
    whole = [i not in cubic and bool(whole_block(C, windows, B * sum(counts[i // 2]), i == 0)) for i in range(n)]
    assert any(whole)
    print("stage of whole blocks", C, B, rows, cols, counts, cubic, flush=True)
    inps = [synth.make_block_inputs(spec, 90 + i, ranges={"a_fc2_in": (-0.07, 0.35)} if i in cubic else None) for i in range(n)]
    x = torch.from_numpy(synth.make_feature_map(spec, 90, blobs=True)).cuda()
    blocks = [gh.GpuBlock(inp, 3 if i % 2 else 0) for i, inp in enumerate(inps)]
    try:
        scores, perm = blocks[0].score_select(x, k_high[0])
        y, tmp = torch.full_like(x, float("nan")), torch.full_like(x, float("nan"))
        s, p = torch.empty_like(scores), torch.full_like(perm, -1)
        ws = blocks[0].ws.fill_(UNTOUCHED)
        M.mixaq_stage_forward([b.blk for b in blocks], x, k_high, k_low, y, tmp, s, p, ws)
        assert _untouched(ws) == (all(whole) and not forks)
        ref = x
        for i, b in enumerate(blocks):
            M.mixaq_block_set_fused(b.blk, 0)
            ref = b.forward_pruned(ref, perm, k_high[i // 2], k_low[i // 2])
        assert torch.equal(s, scores) and torch.equal(p, perm) and torch.equal(y, ref)
    finally:
        for b in blocks:
            b.close()
