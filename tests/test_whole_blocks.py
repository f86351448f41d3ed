"""Blocks of few windows that one kernel takes whole (csrc/block_plan.h) against the separate kernels, bit for bit, and the rule itself."""
import ctypes
import os
import subprocess

import pytest
import torch

from paper_2507_19131_amd import binding as M
from paper_2507_19131_amd import synth
import gpu_harness as gh
from test_kernel_resources import kernels, workgroups_per_cu      # noqa: F401 (a fixture)

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_19131_amd", "csrc")


@pytest.fixture(scope="module")
def whole_block(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text('#include "block_plan.h"\nextern "C" int whole(int C, int w, int n, int scored) { return mixaq::whole_block(C, w, n, scored); }\n')
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-fPIC", "-shared", "-I", CSRC, "-o", str(d / "plan.so"), str(d / "plan.cpp")], check=True)
    return ctypes.CDLL(str(d / "plan.so")).whole


@pytest.mark.parametrize("C", [96, 128, 192, 256, 384, 512, 768, 1024])
def test_only_the_widths_that_have_the_kernel_and_only_what_fits_the_chip_at_once(whole_block, C):
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


# B, rows and columns of windows, pruned share: the smallest, ragged and both ends of each range
MAPS = {96: ((1, 1, 1, 0.0), (3, 3, 5, 0.4), (1, 16, 16, 0.0), (2, 10, 14, 0.2), (1, 16, 22, 0.0), (2, 16, 16, 0.0)),
        128: ((1, 12, 12, 0.0), (1, 16, 16, 0.0), (2, 10, 14, 0.2), (1, 20, 20, 0.0), (2, 16, 16, 0.0)),
        192: ((1, 12, 12, 0.0), (2, 8, 16, 0.0), (2, 10, 14, 0.2))}


@pytest.mark.gpu
@pytest.mark.parametrize("bits", [(8, 4, 8), (8, 2, 4), (4, 8, 8)])
@pytest.mark.parametrize("C,B,rows,cols,pruned", [(C, *m) for C, maps in MAPS.items() for m in maps])
def test_whole_blocks_have_the_bits_of_the_separate_kernels(whole_block, C, B, rows, cols, pruned, bits):
    """Both shifts, given list and scores, both branches' widths packed (2 and 4 bits) and not: whole maps of both forms, and the lists."""
    spec = synth.BlockSpec(B, 7 * rows - 3, 7 * cols - 5, C, C // 32, act_bits_high=bits[0], act_bits_low=bits[1], weight_bits=bits[2])
    n = spec.nW
    k_low = n - n // 3 - int(pruned * n)
    k_high = n // 3 if n > 1 else 1
    k_low = max(0, min(k_low, n - k_high))
    assert n == rows * cols and whole_block(C, B * n, B * (k_high + k_low), 0)
    inp = synth.make_block_inputs(spec, 31 + C)
    x = torch.from_numpy(synth.make_feature_map(spec, 31 + n, blobs=True)).cuda()
    for shift in (0, 3) if min(rows, cols) > 1 else (0,):            # a shift needs two windows either way
        with gh.GpuBlock(inp, shift) as whole, gh.GpuBlock(inp, shift, fused=0) as parts:
            scores, perm = whole.score_select(x, k_high)
            y = parts.forward_pruned(x, perm, k_high, k_low)
            assert not torch.isnan(y).any()
            assert torch.equal(whole.forward_pruned(x, perm, k_high, k_low), y)
            assert torch.equal(whole.forward_pruned(x, None, k_high, k_low), y)


@pytest.mark.gpu
@pytest.mark.parametrize("C,B,rows,cols", [(96, 2, 8, 12), (128, 2, 16, 16), (192, 2, 9, 9)])
def test_stages_of_whole_blocks(C, B, rows, cols):
    """A batch that would run as two chains of the separate forms: map, scores and list as block by block through the separate kernels."""
    spec = synth.BlockSpec(B, 7 * rows, 7 * cols - 2, C, C // 32)
    inps = [synth.make_block_inputs(spec, 90 + i) for i in range(6)]
    x = torch.from_numpy(synth.make_feature_map(spec, 90, blobs=True)).cuda()
    k = spec.nW // 2
    blocks = [gh.GpuBlock(inp, 3 if i % 2 else 0) for i, inp in enumerate(inps)]
    try:
        scores, perm = blocks[0].score_select(x, k)
        y, tmp = torch.empty_like(x), torch.empty_like(x)
        s, p = torch.empty_like(scores), torch.empty_like(perm)
        M.mixaq_stage_forward([b.blk for b in blocks], x, [k] * 3, None, y, tmp, s, p, blocks[0].ws)
        ref = x
        for b in blocks:
            M.mixaq_block_set_fused(b.blk, 0)
            ref = b.forward(ref, perm, k)
        assert torch.equal(s, scores) and torch.equal(p, perm) and torch.equal(y, ref)
    finally:
        for b in blocks:
            b.close()
