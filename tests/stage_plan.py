"""The library's own rules of which stages run as two chains and which images a chain takes when (csrc/stage_plan.h), and of which launches
take a whole block in one kernel (csrc/block_plan.h), built for the host."""
import ctypes
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_19131_amd", "csrc")

_SOURCE = r'''
#include "block_plan.h"
#include "stage_plan.h"
extern "C" {
int splits(int B, int nW) { return mixaq::stage_splits(B, nW); }
int pays(int B, int nW, int C, int blocks) { return mixaq::stage_split_pays(B, nW, C, blocks); }
int rounds(int B, int nW, int C) { return mixaq::stage_rounds(B, nW, C); }
int round_images(int B, int nW, int C, int chain) { return mixaq::round_images(B, nW, C, chain); }
int whole_block(int C, int windows, int computed, int scored) { return mixaq::whole_block(C, windows, computed, scored); }
int whole_stage(int C, int windows, int computed, int blocks) { return mixaq::whole_stage(C, windows, computed, blocks); }
int part_first(int B, int nW, int C, int chain, int round) { return mixaq::stage_part(B, nW, C, chain, round).first; }
int part_images(int B, int nW, int C, int chain, int round) { return mixaq::stage_part(B, nW, C, chain, round).images; }
}
'''


def _build():
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "plan.cpp"), os.path.join(d, "plan.so")
        with open(src, "w") as f:
            f.write(_SOURCE)
        subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-fPIC", "-shared", "-I", CSRC, "-o", so, src], check=True)
        return ctypes.CDLL(so)


lib = _build()


def forks(spec, n_blocks, k_high=None, k_low=None):
    """Whether mixaq_stage_forward runs these blocks as two chains (fused kernels at every block: C <= 384, mlp_ratio 4), by the counts of every
    pair (None: no window is pruned).  Blocks with a table of steps for the GELU and bounded sums; others fork also where this says that
    one chain of blocks in one kernel each is shorter."""
    if not (n_blocks > 1 and spec.C <= 384 and spec.mlp_ratio == 4 and lib.splits(spec.B, spec.nW) and
            lib.pays(spec.B, spec.nW, spec.C, n_blocks)):
        return False
    pairs = (n_blocks + 1) // 2
    computed = [spec.nW] * pairs if k_low is None else [h + l for h, l in zip(k_high, k_low)]
    assert len(computed) == pairs
    return not all(lib.whole_stage(spec.C, spec.B * spec.nW, spec.B * n, n_blocks) for n in computed)


def rounds(spec):
    """In how many rounds the two chains of such a stage go through their images."""
    return lib.rounds(spec.B, spec.nW, spec.C)
