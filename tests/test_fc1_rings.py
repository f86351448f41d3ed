"""The two rings of FC1's 64 x 64 tiles (csrc/product_plan.h) on both sides of the line between them, against the oracle."""
import ctypes
import os
import subprocess

import pytest

from paper_2507_19131_amd import synth
import gpu_harness as gh

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_19131_amd", "csrc")


@pytest.fixture(scope="module")
def ring_of_four(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text('#include "product_plan.h"\nextern "C" int four(int rows, int N) { return mixaq::fc1_ring_of_four(rows, N); }\n')
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-fPIC", "-shared", "-I", CSRC, "-o", str(d / "plan.so"), str(d / "plan.cpp")], check=True)
    return ctypes.CDLL(str(d / "plan.so")).four


@pytest.mark.parametrize("C,two", [(512, 1024), (768, 640), (1024, 512)])
def test_the_line(ring_of_four, C, two):
    """Two 64 x 64 tiles a CU; rows come in whole 128s."""
    assert not ring_of_four(two, 4 * C) and ring_of_four(two + 128, 4 * C)


# rows of windows, columns, kept in the high branch, a range narrow enough that the GELU has no table of steps
@pytest.mark.gpu
@pytest.mark.parametrize("narrow", [False, True])
@pytest.mark.parametrize("C,rows,cols,high,four", [(512, 2, 9, 9, False), (512, 3, 8, 24, True), (512, 4, 6, 11, True), (768, 3, 4, 12, False),
                                                   (768, 3, 5, 15, True), (1024, 2, 4, 8, False), (1024, 2, 5, 4, True)])
def test_blocks_on_both_sides_of_the_line(ring_of_four, C, rows, cols, high, four, narrow):
    spec = synth.BlockSpec(1, 7 * rows, 7 * cols - 1, C, C // 32)
    padded = sum(-(-49 * n // 128) * 128 for n in (high, spec.nW - high))
    assert ring_of_four(padded, 4 * C) == four
    inp = synth.make_block_inputs(spec, 7 + C, ranges={"a_fc2_in": (-0.07, 0.35)} if narrow else None)
    gh.assert_parity(gh.compare_block(inp, synth.make_feature_map(spec, 7, blobs=True), high, taps=("acc_fc1", "a_fc2_in", "acc_fc2")))
