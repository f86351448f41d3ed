"""What bench.py says about the form of a stage call against the library's own rules (csrc/stage_plan.h, csrc/block_plan.h).  CPU only."""
import pytest

import bench
import stage_plan
from paper_2507_19131_amd import synth


@pytest.mark.parametrize("C", [96, 128, 192, 256, 384, 512, 768, 1024])
def test_two_chains_and_blocks_in_one_kernel(C):
    for nW in list(range(1, 530)) + [1392, 2047, 2049, 4096]:
        for B in (1, 2, 3, 4, 9):
            spec = synth.BlockSpec(B, 7, 7 * nW, C, C // 32)
            assert bench.whole_block(C, B * nW) == bool(stage_plan.lib.whole_block(C, B * nW, B * nW, 0)) == bool(stage_plan.lib.whole_block(C, B * nW, B * nW, 1))
            for blocks in (1, 2, 6, 7, 8, 9, 12, 13, 24):
                assert bench.two_chains(B, B * nW, C, blocks) == stage_plan.forks(spec, blocks), (B, nW, blocks)
