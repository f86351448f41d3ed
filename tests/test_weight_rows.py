"""Rows of weight codes and the bound of the integer sums over them (csrc/weight_rows.h), compiled for the host.  CPU only."""
import os
import subprocess
import textwrap

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2507_19131_amd", "csrc")

PROGRAM = textwrap.dedent(r'''
    #include <cstdio>
    #include <cstdlib>
    #include <cstring>
    #include <vector>
    #include "weight_rows.h"
    using namespace mixaq;
    int main(int argc, char** argv)
    {
        if (!strcmp(argv[1], "fit")) { printf("%d\n", sums_fit(atoi(argv[2]), atoi(argv[3]), atoi(argv[4]), atoi(argv[5]))); return 0; }
        const int K = atoi(argv[2]);
        std::vector<int8_t> w(K);
        while (fread(w.data(), 1, K, stdin) == (size_t)K) {
            const RowCodes c = row_codes(w.data(), K);
            printf("%d %d %d %d\n", c.sum, c.width, c.lowest, c.highest);
        }
        return 0;
    }
''')


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("weight_rows")
    src, exe = d / "rows.cpp", d / "rows"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O3", "-std=c++17", "-fsanitize=undefined", "-fno-sanitize-recover", "-I", CSRC, "-o", str(exe), str(src)], check=True)
    return lambda args, data=b"": subprocess.run([str(exe)] + [str(a) for a in args], input=data, check=True, capture_output=True).stdout.decode()


@pytest.mark.parametrize("K", [1, 15, 16, 33, 96, 768, 8192])
def test_sum_width_and_extremes_of_a_row(program, K):
    rng = np.random.default_rng(K)
    rows = [np.full(K, v) for v in (-128, 127, 0, -1)] + [rng.integers(-128, 128, K), rng.integers(-2, 2, K), rng.integers(-8, 1, K)]
    for at in (0, K // 2, K - 1):                          # one code out of a 4-bit range
        for v in (-9, 8, -128, 127):
            row = rng.integers(-8, 8, K)
            row[at] = v
            rows.append(row)
    w = np.array(rows, dtype=np.int8)
    got = np.array([[int(v) for v in line.split()] for line in program(["rows", K], w.tobytes()).splitlines()])
    i = w.astype(np.int64)
    want = np.stack([i.sum(1), np.abs(i).sum(1), i.min(1), i.max(1)], axis=1)
    assert np.array_equal(got, want)


@pytest.mark.parametrize("bits", [2, 4, 8])
@pytest.mark.parametrize("zp_at", ["low", "middle", "high"])
def test_sums_fit_up_to_the_bound_and_not_beyond(program, bits, zp_at):
    """The largest sum of a row of that width is reached with every code at the end farther from the zero point."""
    qmin, qmax = -(1 << (bits - 1)), (1 << (bits - 1)) - 1
    zp = {"low": qmin, "middle": 0, "high": qmax}[zp_at]
    reach = max(qmax - zp, zp - qmin)
    widest = (2**22 - 1) // reach                          # widest * reach < 2^22 <= (widest + 1) * reach
    fits = lambda width: int(program(["fit", width, qmin, qmax, zp]))
    assert fits(widest) == 1 and fits(widest + 1) == 0
    assert fits(0) == 1 and fits(2**31 - 1) == 0
