"""Evaluation points: the paths chosen by the number of points (one or two
streams from 50,000 on, with the derivative descents up to 8192 points and the
leaves' own kernel above), the scan over one block or several (trees of more
than 8192 boxes), ragged targets per leaf, lists of more than 64 boxes.

The same points evaluated in calls on either side of a line agree to rounding
(FP64 1e-12, the parity bar; mixed precision 1e-6, or where one lane sums a
whole leaf of n sources in FP32 the random-walk rounding 2^-24 sqrt(n) of each
side if that is more), and a sample agrees with
the direct sum to the truncation of the order (0.5^p and a constant: 1e-7 at
p = 30 is generous)."""
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


@pytest.mark.parametrize("prec,bar", [("fp64", 1e-12), ("mixed", 1e-6)])
@pytest.mark.parametrize("n,L,M", [(1001, 4, 8193), (40000, 7, 50001), (70001, 8, 9000), (3000, 1, 8200), (500, 2, 60000)])
def test_paths_agree(F, orc, prec, bar, n, L, M):
    if prec == "mixed":
        bar = max(bar, 2 * 2.0 ** -24 * np.sqrt(n / 4 ** (L - 1)))
    z, m, _ = W.uniform(n, seed=n)
    y = W.uniform(M, seed=n + 1)[0]
    y[::97] = 1.5 + 0.3j + 1e-3 * y[::97]          # some outside every disc, a leaf's worth together
    pl = F.plan(F.build_tree(dev(z), L), 30, 0.5, prec)
    md = dev(m)
    phi, dphi = (host(x) for x in F.evaluate_points(pl, md, dev(y), field=True))
    part = slice(0, min(M, 5000))                  # descents, one stream
    a, b = (host(x) for x in F.evaluate_points(pl, md, dev(y[part]), field=True))
    assert e2(phi[part], a) <= bar and e2(dphi[part], b) <= bar
    plain = host(F.evaluate_points(pl, md, dev(y)))
    assert e2(plain, phi) <= bar
    sub = np.arange(0, M, max(1, M // 500))
    assert e2(phi[sub], orc.direct_points(z, m, y[sub])) <= max(bar, 1e-7)
    assert e2(dphi[sub], orc.direct_deriv_points(z, m, y[sub])) <= max(bar, 1e-7)


def test_long_lists(F, orc):
    # a point far from a cluster: strong lists of more than 64 boxes
    rng = np.random.default_rng(2)
    z = np.concatenate([rng.random(20000) + 1j * rng.random(20000), [300.0 + 200.0j, -150.0 - 400.0j]])
    m = rng.standard_normal(z.size) + 1j * rng.standard_normal(z.size)
    y = np.concatenate([rng.random(9000) + 1j * rng.random(9000), z[-2:] + 0.5])
    pl = F.plan(F.build_tree(dev(z), 6), 30, 0.5, "fp64")
    phi, dphi = (host(x) for x in F.evaluate_points(pl, dev(m), dev(y), field=True))
    assert e2(phi, orc.direct_points(z, m, y)) <= 1e-7
    assert e2(dphi, orc.direct_deriv_points(z, m, y)) <= 1e-7
