"""Leaves of many points where the near field runs on the second stream and gathers
the strengths itself (more than 64 points per leaf), and its neighbours: one
stream below 16,385 points with split lists and below 2049 points with more than 32
terms.  Every form of the evaluation against the direct sum (converged orders;
1e-12 FP64, 1e-6 mixed) and against each other to the bit."""
import numpy as np
import pytest

from paper_1311_1006_amd import workloads as W

from gpu_util import dev, e2, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,bar", [("fp64", 1e-12), ("mixed", 1e-6)])
@pytest.mark.parametrize("n,L,p", [(2048, 3, 44), (2049, 3, 44), (9000, 4, 48), (2049, 2, 64), (16384, 4, 46),
                                   (16385, 4, 32), (33000, 6, 46)])
def test_evaluations_agree(orc, prec, bar, n, L, p):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1311_1006_amd as F
    z, m, _ = W.uniform(n, seed=n + p)
    tree, md = F.build_tree(dev(z), L), dev(m)
    pl = F.plan(tree, p, 0.5, prec)
    phi = host(F.evaluate(pl, md))                     # lists pending
    sub = np.arange(0, n, max(1, n // 2000))
    # 32 terms leave 2^-32 and a constant
    assert e2(phi[sub], orc.direct_points(z, m, z[sub])) <= (bar if p > 32 else max(bar, 1e-8))
    assert np.array_equal(host(F.evaluate(pl, md)), phi)
    out = dev(np.zeros(n, np.complex128))
    F.evaluate_static(pl, md, out)
    assert np.array_equal(host(out), phi)
    g = F.plan(tree, p, 0.5, prec, graph=True)
    gout = dev(np.zeros(n, np.complex128))
    other = dev(m[::-1])
    for _ in range(3):                                 # replays, eager work of other strengths between
        gout.zero_()
        F.evaluate(g, md, gout)
        F.evaluate(pl, other)
        assert np.array_equal(host(gout), phi)
    near, far = F.evaluate_parts(pl, md)
    assert e2(host(near) + host(far), phi) <= 1e-15
