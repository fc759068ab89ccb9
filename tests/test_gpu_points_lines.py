"""Evaluation points with the derivative on both sides of the line between descents
and the leaves' own kernel (8192 points, or 3 per leaf in FP64 and 2 in mixed
precision if that is more), on one stream and on two: the same points in one call
and in calls of 5000 (always descents) agree to rounding, and a sample agrees
with the direct sum to the truncation (0.5^30 and a constant: 1e-7)."""
import numpy as np
import pytest

from paper_1311_1006_amd import workloads as W

from gpu_util import dev, e2, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,bar", [("fp64", 1e-12), ("mixed", 1e-6)])
@pytest.mark.parametrize("n,L,M", [(70001, 8, 32768), (70001, 8, 32769), (70001, 8, 49152), (70001, 8, 49153),
                                   (300001, 9, 100000)])
def test_points_at_the_line(orc, prec, bar, n, L, M):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1311_1006_amd as F
    z, m, _ = W.uniform(n, seed=n)
    y = W.uniform(M, seed=n + 1)[0]
    y[::97] = 1.5 + 0.3j + 1e-3 * y[::97]          # some outside every disc
    pl = F.plan(F.build_tree(dev(z), L), 30, 0.5, prec)
    md = dev(m)
    phi, dphi = (host(x) for x in F.evaluate_points(pl, md, dev(y), field=True))
    part = slice(M - 5000, M)
    a, b = (host(x) for x in F.evaluate_points(pl, md, dev(y[part]), field=True))
    assert e2(phi[part], a) <= bar and e2(dphi[part], b) <= bar
    sub = np.arange(0, M, M // 500)
    assert e2(phi[sub], orc.direct_points(z, m, y[sub])) <= max(bar, 1e-7)
    assert e2(dphi[sub], orc.direct_deriv_points(z, m, y[sub])) <= max(bar, 1e-7)


@pytest.mark.parametrize("prec,bar", [("fp64", 1e-12), ("mixed", 1e-6)])
@pytest.mark.parametrize("n,L", [(20000, 6), (70001, 7)])
def test_points_in_leaves_with_long_lists(orc, prec, bar, n, L):
    # three sources far off: their leaf is strong with every leaf of the level (more
    # than 512 boxes, so that its points are descended), the others' lists are short
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1311_1006_amd as F
    rng = np.random.default_rng(n)
    z, m, _ = W.uniform(n, seed=n)
    far = rng.integers(0, n, 3)
    z[far] = 300.0 * np.exp(2j * np.pi * rng.random(3))
    y = W.uniform(20001, seed=n + 1)[0]
    y[::9] = z[rng.integers(0, n, y[::9].size)] + 1e-4
    y[:30] = z[far][np.arange(30) % 3] + 0.1 * rng.random(30)
    pl = F.plan(F.build_tree(dev(z), L), 30, 0.5, prec)
    off, _ = pl.download_list(0, L - 1, 0)
    assert np.diff(off).max() > 512
    md = dev(m)
    phi, dphi = (host(x) for x in F.evaluate_points(pl, md, dev(y), field=True))
    part = slice(0, 5000)
    a, b = (host(x) for x in F.evaluate_points(pl, md, dev(y[part]), field=True))
    assert e2(phi[part], a) <= bar and e2(dphi[part], b) <= bar
    sub = np.concatenate([np.arange(30), np.arange(30, y.size, 50)])
    assert e2(phi[sub], orc.direct_points(z, m, y[sub])) <= max(bar, 1e-7)
    assert e2(dphi[sub], orc.direct_deriv_points(z, m, y[sub])) <= max(bar, 1e-7)
    assert e2(phi[:30], orc.direct_points(z, m, y[:30])) <= 10 * max(bar, 1e-7)


@pytest.mark.parametrize("prec,bar", [("fp64", 1e-12), ("mixed", 1e-6)])
@pytest.mark.parametrize("M", [32768, 32769])
def test_points_beside_clusters_at_the_line_of_the_lists(orc, prec, bar, M):
    # 32 points per leaf: leaves with more than 64 boxes in their lists are
    # descended up to there, with more than 512 above it
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1311_1006_amd as F
    z, m = W.clustered(30000, seed=7)[:2]
    rng = np.random.default_rng(M)
    y = W.uniform(M, seed=8)[0]
    y[::3] = z[rng.integers(0, z.size, y[::3].size)] + 1e-4
    pl = F.plan(F.build_tree(dev(z), 6), 30, 0.5, prec)
    cnt = np.diff(pl.download_list(0, 5, 0)[0])
    assert (cnt > 64).any() and (cnt <= 64).any()
    md = dev(m)
    phi, dphi = (host(x) for x in F.evaluate_points(pl, md, dev(y), field=True))
    part = slice(M - 5000, M)
    a, b = (host(x) for x in F.evaluate_points(pl, md, dev(y[part]), field=True))
    assert e2(phi[part], a) <= bar and e2(dphi[part], b) <= bar
    sub = np.arange(0, M, M // 500)
    assert e2(phi[sub], orc.direct_points(z, m, y[sub])) <= max(bar, 1e-7)
    assert e2(dphi[sub], orc.direct_deriv_points(z, m, y[sub])) <= max(bar, 1e-7)
