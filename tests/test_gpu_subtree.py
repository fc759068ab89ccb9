"""The far field's upward and downward passes by subtrees: problems of unlike
depth in one tree (one and two levels, which have no shifts between levels,
and deeper ones), and trees deep enough for several launches per pass in the
direct and in the staged form.

FP64 against the oracle's serial FMM at equal (p, theta, N_levels): relative
2-norm <= 1e-12, the bar of the other parity tests (both truncate the same
series; what differs is rounding); at p >= 40, where the unscaled operators of
the oracle's FMM overflow on small boxes, against its direct sum (the
truncation, about 0.5^p, is below the bar).  A problem of a batch of unlike depths has
the bits it has alone with levelwise=True (the same staged kernels)."""
import numpy as np
import pytest

from paper_1311_1006_amd import workloads as W

from gpu_util import dev, e2, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1311_1006_amd as F
    F.lib()
    return F


def reference(orc, z, m, p, L):
    return orc.direct(z, m) if p >= 40 else orc.fmm(z, m, p, 0.5, L)


@pytest.mark.parametrize("p", [5, 16, 17, 33, 64])
def test_problems_of_unlike_depth(orc, F, p):
    Ls = [1, 2, 3, 5, 7, 8]
    zs, ms = zip(*[W.uniform(n, seed=n + p)[:2] for n in (60, 70, 901, 4001, 30011, 40009)])
    off = np.concatenate([[0], np.cumsum([len(z) for z in zs])]).tolist()
    tree = F.build_tree(dev(np.concatenate(zs)), Ls, offsets=off)
    md = dev(np.concatenate(ms))
    phi = host(F.evaluate(F.plan(tree, p, 0.5, "fp64"), md))
    mixed = host(F.evaluate(F.plan(tree, p, 0.5, "mixed"), md))
    for b, L in enumerate(Ls):
        sl = slice(off[b], off[b + 1])
        ref = reference(orc, zs[b], ms[b], p, L)
        assert e2(phi[sl], ref) <= 1e-12
        if L >= 3:
            tb, mb = F.build_tree(dev(zs[b]), L), dev(ms[b])
            np.testing.assert_array_equal(phi[sl], host(F.evaluate(F.plan(tb, p, 0.5, "fp64", levelwise=True), mb)))
            np.testing.assert_array_equal(mixed[sl], host(F.evaluate(F.plan(tb, p, 0.5, "mixed", levelwise=True), mb)))


@pytest.mark.parametrize("levelwise", [False, True])
@pytest.mark.parametrize("L,p", [(10, 12), (9, 40)])
def test_deep_trees(orc, F, L, p, levelwise):
    # L = 10: three upward launches and two staged ones (p <= 32); L = 9 at
    # p = 40: levels two at a time
    z, m, _ = W.uniform(4 ** (L - 1) + 1001, seed=L)
    pl = F.plan(F.build_tree(dev(z), L), p, 0.5, "fp64", levelwise=levelwise)
    assert e2(host(F.evaluate(pl, dev(m))), reference(orc, z, m, p, L)) <= 1e-12
