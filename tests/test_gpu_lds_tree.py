"""The in-LDS tree stage at the edges of its forms, against the oracle's tree to
the bit: segments of 1, 2 and 4 points per thread (1024, 2048, 4096 points), four
workgroups per segment and one (more than 64 segments), the positions read by
the stage itself (no global stage) and after an even and an odd number of
global stages, densities that take the finer buckets, and boxes without extent
(their scaling radius is an ancestor's, from this or from a global stage)."""
import numpy as np
import pytest

from gpu_util import dev, host, same_tree

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1311_1006_amd as F
    F.lib()
    return F


def points(kind, n, rng):
    if kind == "power":         # dense towards 0 in both coordinates
        return rng.random(n) ** 6 + 1j * rng.random(n) ** 6
    if kind == "half":          # half of the points at one place: boxes without extent at many levels
        z = rng.random(n) + 1j * rng.random(n)
        z[rng.permutation(n)[:n // 2]] = 0.75 + 0.125j
        return z
    return rng.random(n) + 1j * rng.random(n)


@pytest.mark.parametrize("kind", ["uniform", "power", "half"])
@pytest.mark.parametrize("n,L", [(1, 1), (4, 2), (1023, 3), (1024, 2), (1025, 2), (1025, 3), (2048, 4), (2049, 5),
                                 (4096, 3), (4097, 4), (8193, 5), (16385, 6), (40000, 3), (262143, 8), (300001, 8)])
def test_lds_tree_forms(orc, F, kind, n, L):
    same_tree(orc, F, points(kind, n, np.random.default_rng(n + L)).astype(np.complex128), L)


def test_small_batch_reads_its_positions(orc, F):
    # no problem has a global stage: several segments of unlike size, then one
    # of them with a position that is not finite
    rng = np.random.default_rng(5)
    sizes, L = [5, 4096, 1000, 64, 2049], [2, 4, 3, 4, 5]
    off = np.concatenate([[0], np.cumsum(sizes)])
    zs = [points("half" if i % 2 else "uniform", n, rng) for i, n in enumerate(sizes)]
    z = np.concatenate(zs).astype(np.complex128)
    tree = F.build_tree(dev(z), L, offsets=off.tolist())
    for b, (zb, lb) in enumerate(zip(zs, L)):
        perm, rng_g, geom = tree.download(b)
        perm_o, rng_o, geom_o = orc.tree(zb.astype(np.complex128), lb)
        assert np.array_equal(geom.view(np.uint64), geom_o.view(np.uint64)), b
    bad = z.copy()
    bad[off[2] + 3] = complex(0.5, np.inf)
    with pytest.raises(F.FmmError):
        F.build_tree(dev(bad), L, offsets=off.tolist()).download(0)
    F.build_tree(dev(z), L, offsets=off.tolist()).download(0)


@pytest.mark.parametrize("n,L", [(1000, 4), (9000, 5), (30000, 6)])
def test_evaluation_with_boxes_without_extent(orc, F, n, L):
    # a quarter of the points at one place: boxes without
    # extent take an ancestor's scaling radius; the parity bar, 1e-12
    rng = np.random.default_rng(n)
    z = points("uniform", n, rng).astype(np.complex128)
    k = n // 4
    z[rng.permutation(n)[:k]] = z[0]
    m = rng.standard_normal(n) + 0j
    phi = host(F.evaluate(F.plan(F.build_tree(dev(z), L), 17, 0.5, "fp64"), dev(m)))
    ref = orc.fmm(z, m, 17, 0.5, L)
    assert np.linalg.norm(phi - ref) <= 1e-12 * np.linalg.norm(ref)
