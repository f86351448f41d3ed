"""GELU and the quantizer of its output as a table of steps (csrc/gelu_steps.h), compiled for the host and compared with the
oracle's own GELU and quantizer.  CPU only."""
import os
import subprocess
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2507_19131_amd", "csrc")

PROGRAM = textwrap.dedent(r'''
    #include <cstdio>
    #include <cstdlib>
    #include <random>
    #include <cmath>
    #include <algorithm>
    static long fma_calls = 0;
    static inline float counted_fma(float a, float b, float c) { ++fma_calls; return __builtin_fmaf(a, b, c); }
    #define fmaf counted_fma
    #include "gelu_steps.h"
    #undef fmaf
    #include "arith.h"
    using namespace mixaq;
    int main(int argc, char** argv)
    {
        const float lo = atof(argv[1]), hi = atof(argv[2]);
        const int bits = atoi(argv[3]), qmin = -(1 << (bits - 1)), qmax = -qmin - 1;
        const float s = (hi - lo) / ((1 << bits) - 1);
        const int zp = (int)std::min(std::max(std::rint(qmin - lo / s), (float)qmin), (float)qmax);
        float cubic[ORC_GELU_INTERVALS * 4];
        for (int e = 0; e < ORC_GELU_INTERVALS * 4; ++e) cubic[e] = orc_gelu_tab[e / 4][e % 4] * 16.0f;
        const float inv = 1.0f / s;
        GeluSteps t;
        if (!t.build(cubic, ORC_GELU_INTERVALS, inv / 16.0f, GELU_STEP_MAGIC + zp, GELU_STEP_MAGIC + qmin, GELU_STEP_MAGIC + qmax)) { printf("none\n"); return 0; }
        const long built = fma_calls;
        long wrong = 0, seen = 0;
        auto check = [&](float x) { ++seen; wrong += t.looked_up(16.0f * x) != orc_q(orc_gelu_pinned(x), inv, zp, bits); };
        auto around = [&](float x, int n) {
            float up = x, down = x;
            for (int k = 0; k < n; ++k) { check(up); check(down); up = nextafterf(up, INFINITY); down = nextafterf(down, -INFINITY); }
        };
        for (float x : {0.0f, -0.0f, INFINITY, -INFINITY, 3e38f, -3e38f, 1e20f, -1e20f, 1e-38f, -1e-38f, 1e-45f, -1e-45f}) check(x / (fabsf(x) > 1e37f && !std::isinf(x) ? 32.0f : 1.0f));
        std::mt19937 gen(5);
        std::normal_distribution<float> wide(0.0f, 4.0f), narrow(0.0f, 0.4f);
        for (int k = 0; k < 300000; ++k) { check(wide(gen)); check(narrow(gen)); check(hi * 1.2f * (gen() * 0x1p-32f)); }
        // every step from both sides, found here from the oracle; and both ends of every entry
        float prev = -6.5f;
        const float end = std::max(hi * 1.1f, 1.0f) + 0.5f;
        for (int k = 1; k <= 60000; ++k) {
            const float x = -6.5f + (end + 6.5f) * k / 60000;
            auto code = [&](float v) { return orc_q(orc_gelu_pinned(v), inv, zp, bits); };
            if (code(x) != code(prev)) {
                float a = prev, b = x;
                while (nextafterf(a, b) != b) { const float m = a + (b - a) / 2; if (m == a || m == b) break; (code(m) == code(prev) ? a : b) = m; }
                around(a, 40);
            }
            prev = x;
        }
        const int spans = (int)(t.index.span / 8);
        for (int i = 1; i <= spans; ++i) around((((i - 0.0625f) / spans) - t.index.offset) / t.index.scale / 16.0f, 60);
        int steps = 0;
        for (int i = 1; i <= spans; ++i) steps += t.table[i].addend < 0x1p99f && t.table[i].factor != t.table[i - 1].factor;
        printf("entries %d pieces %zu seen %ld wrong %ld fma %ld steps %d\n", spans + 1, t.table.size() / 128, seen, wrong, built, steps);
        return 0;
    }
''')


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("gelu_steps")
    src, exe = d / "steps.cpp", d / "steps"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-fsanitize=undefined", "-fno-sanitize-recover", "-I", CSRC,
                    "-I", os.path.join(ROOT, "oracle"), "-o", str(exe), str(src)], check=True)
    return lambda *a: subprocess.run([str(exe)] + [str(v) for v in a], check=True, capture_output=True, text=True).stdout.split()


@pytest.mark.parametrize("lo,hi,bits", [(-0.17, 0.8, 8), (-0.159375, 0.75, 4), (-0.17, 0.8, 2), (-0.159375, 0.75, 3), (-0.17, 4.0, 8),
                                        (-0.17, 50.0, 8), (-0.17, 2000.0, 8), (0.0, 0.5, 4), (-0.17, 0.0, 5), (-1.0, 1.0, 6), (-0.3, 1.3, 7), (5.0, 9.0, 2)])
def test_codes_by_steps_are_the_pinned_codes(program, lo, hi, bits):
    out = program(lo, hi, bits)
    assert out[0] == "entries" and 2 <= int(out[1]) <= 1664 and int(out[3]) <= 13
    assert int(out[5]) > 900000 and int(out[7]) == 0


@pytest.mark.parametrize("lo,hi", [(-0.17, 0.8), (-0.17, 4.0), (-0.17, 50.0)])
def test_a_step_is_found_from_the_two_before_it(program, lo, hi):
    """The builder runs whenever a block is created.  Walking the neighbours of a step until the value is out of the roundings' reach
    takes about eight evaluations of four fused multiply-adds on each of its two sides, finding it nine more: 100 in all."""
    out = program(lo, hi, 8)
    fma, steps = int(out[9]), int(out[11])
    assert steps >= 250 and fma <= 120 * steps, out


@pytest.mark.parametrize("lo,hi,bits", [(-0.07, 0.35, 8),                         # steps too close for the table
                                        ("-0x1.5f989ep-3", "0x1.5ea916p+2", 8),   # a code that returns beyond its step
                                        (-1e30, 1e31, 8), (-1e-20, 1e-20, 4)])
def test_quantizers_without_a_table(program, lo, hi, bits):
    assert program(lo, hi, bits) == ["none"]
