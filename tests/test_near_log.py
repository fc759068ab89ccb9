"""The logarithm of the FP64 logarithmic near field (csrc/near_log.h), value by
value on the CPU against 113-bit arithmetic: the table's intervals and their
edges, the neighbourhood of 1, near-field distances and the whole exponent range.

The bound, in units in the last place of the result: 0.5 for the last rounding;
the economised term leaves at most 2^-57 of the result (1/16 unit); the series'
own roundings and the truncated low part of log c are below 2^-6 unit each: 0.6.
The root mean square of a well-rounded value is 1/sqrt(12) = 0.289; with a tenth
of a unit added at most: 0.31."""
import math
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "near_log.h"
#include <cstdio>
#include <functional>
#include <random>
#include <quadmath.h>
struct D2 { double x, y; };
int main()
{
    D2 tab[fmm::kLogTab];
    fmm::log_table(tab);
    std::mt19937_64 g(1);
    std::uniform_real_distribution<double> U(0, 1);
    auto run = [&](const char* name, int n, const std::function<double(int)>& gen) {
        double mx = 0, s2 = 0;
        for (int i = 0; i < n; ++i) {
            const double x = gen(i), v = fmm::half_log(x, tab);
            const __float128 ref = logq((__float128)x) / 2;
            const double d = std::fabs((double)ref);
            if (d == 0) { if (v != 0) mx = 1e9; continue; }
            const double e = std::fabs((double)(((__float128)v - ref) / (std::nextafter(d, INFINITY) - d)));
            s2 += e * e;
            mx = std::fmax(mx, e);
        }
        std::printf("%s %.6f %.6f\n", name, mx, std::sqrt(s2 / n));
    };
    const int n = 150000;
    run("intervals", n, [&](int) { return 0.75 + 0.75 * U(g); });
    run("near-one", n, [&](int) { return 1 + 0.04 * (U(g) - 0.5); });
    run("at-one", n, [&](int) { return 1 + (U(g) - 0.5) * std::exp2(-50 * U(g)); });
    run("exponents", n, [&](int) { return std::exp(1400 * U(g) - 700); });
    run("distances", n, [&](int) { return std::exp(std::log(1e-12) * U(g)); });
    run("edges", 129 * 41 * 3, [&](int i) {
        const int k = i % 129, st = (i / 129) % 41 - 20;
        double x = k < 64 ? 0.75 + k / 256.0 : 1 + (k - 64) / 128.0;
        for (int q = 0; q < std::abs(st); ++q) x = std::nextafter(x, st > 0 ? 4 : 0);
        return x * std::exp2((double)((i / 129 / 41) % 3 - 1));
    });
    const double inf = INFINITY;
    std::printf("limits %.17g %.17g %.17g\n", fmm::half_log(inf, tab), fmm::half_log(0x1p-1022, tab),
                fmm::half_log(0x1.fffffffffffffp1023, tab));
}
"""


def test_error_in_units_of_the_result(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    src = tmp_path / "near_log.cpp"
    src.write_text(PROGRAM)
    exe = str(tmp_path / "near_log")
    subprocess.run(["g++", "-O2", "-std=gnu++17", "-ffp-contract=off",
                    "-I" + os.path.join(ROOT, "paper_1311_1006_amd", "csrc"), str(src), "-o", exe, "-lquadmath"],
                   check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split("\n")
    seen = 0
    for line in out:
        f = line.split()
        if len(f) == 3:
            assert float(f[1]) <= 0.6 and float(f[2]) <= 0.31, line
            seen += 1
    assert seen == 6
    lim = [l.split()[1:] for l in out if l.startswith("limits")][0]
    assert lim[0] == "inf"
    for got, x in ((lim[1], sys.float_info.min), (lim[2], sys.float_info.max)):
        assert abs(float(got) - math.log(x) / 2) <= math.ulp(354.0)
