"""The buckets of the in-LDS sort (csrc/lds_bucket.h) on the CPU: monotone in the
coordinate, and after the second level as well filled for a density that crowds
towards its largest coordinate as for its mirror image, in every bucket the last
one included.

n points u^3 (or 1 - u^3), u uniform, in n buckets: the crowded one holds about
n^(2/3) of them, and after the second level n^(4/9): 40 of 4096, 22 of 1000, a few
standard deviations below the 64 up to which a bucket is ranked without a sort."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "lds_bucket.h"
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>
// largest population of a bucket, first level and second; -1: not monotone
static void fill(std::vector<double> c, int nb, int* first, int* second)
{
    std::sort(c.begin(), c.end());
    const double lo = c.front(), ext = c.back() - lo;
    double scale = ext > 0.0 ? nb / ext : 0.0;
    scale = scale < 1e300 ? scale : 0.0;
    std::vector<int> cnt(nb + 1, 0), end(nb + 1, 0);
    std::vector<fmm::LdsPlace> at;
    for (double x : c) at.push_back(fmm::lds_place(x, lo, scale, nb));
    for (auto& a : at) {
        if (a.bucket < 0 || a.bucket >= nb || !(a.place >= 0.0 && a.place <= 1.0)) std::exit(1);
        ++cnt[a.bucket];
    }
    *first = *std::max_element(cnt.begin(), cnt.end());
    std::vector<int> start(nb + 1, 0), fine(c.size(), 0);
    for (int b = 0; b < nb; ++b) start[b + 1] = start[b] + cnt[b];
    int last = -1;
    for (auto& a : at) {
        const int k = fmm::lds_finer(a.place, start[a.bucket], start[a.bucket + 1]);
        if (k < start[a.bucket] || k >= start[a.bucket + 1] || k < last) std::exit(2);
        last = k;
        ++fine[k];
    }
    *second = *std::max_element(fine.begin(), fine.end());
}
int main()
{
    std::mt19937_64 g(7);
    std::uniform_real_distribution<double> U(0, 1);
    for (int n : {1, 2, 1000, 4096})
        for (int kind = 0; kind < 5; ++kind) {
            std::vector<double> c(n);
            for (double& x : c) {
                const double u = U(g);
                x = kind == 0 ? u : kind == 1 ? u * u * u : kind == 2 ? 1 - u * u * u
                  : kind == 3 ? 0.25 : (u < 0.5 ? -1e308 : 1e308);
            }
            int a, b;
            fill(c, (n + 1023) / 1024 * 1024, &a, &b);
            std::printf("%d %d %d %d\n", n, kind, a, b);
        }
}
"""


def test_buckets(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    src, exe = tmp_path / "lds_bucket.cpp", str(tmp_path / "lds_bucket")
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off",
                    "-I" + os.path.join(ROOT, "paper_1311_1006_amd", "csrc"), str(src), "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split("\n")
    fill = {tuple(map(int, l.split()[:2])): tuple(map(int, l.split()[2:])) for l in out if l}
    assert len(fill) == 20
    for n in (1000, 4096):
        assert fill[n, 3] == (n, n)                    # ties: no division separates them
        low, high = fill[n, 1], fill[n, 2]
        assert low[0] > 64 and high[0] > 64            # one crowded bucket of the first level
        assert low[1] <= 64 and high[1] <= 64, (low, high)
