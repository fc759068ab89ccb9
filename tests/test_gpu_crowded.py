"""The in-LDS tree stage on segments whose coordinates crowd into few value
buckets, where it ranks inside larger buckets (up to 64 points) or runs the
merge sort: the oracle's tree, to the bit.  Sizes around a thread's four, a
wavefront's 256 and a segment's 4096 entries; ties, rows of a grid, one tight
cluster, and points of equal coordinates (ordered by input index)."""
import numpy as np
import pytest

from paper_1311_1006_amd import workloads as W

from gpu_util import dev, e2, host, same_tree

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1311_1006_amd as F
    F.lib()
    return F


def points(kind, n, rng):
    if kind == "rows":          # every row and column of the grid in one bucket
        k = int(np.ceil(np.sqrt(n)))
        i = rng.permutation(k * k)[:n]
        return (i % k + 1e-7 * rng.standard_normal(n)) + 1j * (i // k + 1e-7 * rng.standard_normal(n))
    if kind == "cluster":       # all points but one in one bucket
        z = 1e-6 * (rng.standard_normal(n) + 1j * rng.standard_normal(n))
        z[rng.integers(n)] = 1.0 + 1.0j
        return z
    if kind == "ties":          # at most 7 x 3 distinct positions, both signs and zero
        return (rng.integers(-3, 4, n) + 0.0) + 1j * (rng.integers(-1, 2, n) + 0.0)
    return np.full(n, 0.25 - 2.0j)


@pytest.mark.parametrize("kind", ["rows", "cluster", "ties", "equal"])
@pytest.mark.parametrize("n,L", [(16, 2), (65, 3), (257, 4), (1000, 4), (1025, 5), (4095, 6), (4096, 6), (4097, 6),
                                 (20011, 6)])
def test_crowded_segments(orc, F, kind, n, L):
    z = points(kind, n, np.random.default_rng(n))
    same_tree(orc, F, z.astype(np.complex128), L)


@pytest.mark.parametrize("L", [6, 7, 5])
def test_evaluation_on_crowded_segments(orc, F, L):
    # tight clusters (split lists, merge-sorted segments), order 17: the bars of
    # the clustered parity tests, 1e-12 against the oracle's FMM and in mixed
    # precision 1e-6 against the direct sum
    z, m = W.clustered(59000, seed=3, nclusters=16)
    tree, md = F.build_tree(dev(z), L), dev(m)
    ref = orc.fmm(z, m, 17, 0.5, L)
    assert e2(host(F.evaluate(F.plan(tree, 17, 0.5, "fp64"), md)), ref) <= 1e-12
    for theta, p in ((0.5, 17), (0.45, 15)):
        phi = host(F.evaluate(F.plan(tree, p, theta, "mixed"), md))
        sub = W.subsample(z.size, 800, seed=L)
        assert e2(phi[sub], orc.direct(z, m, sub)) <= 1e-6
