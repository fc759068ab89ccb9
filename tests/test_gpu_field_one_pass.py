"""evaluate_field's one-pass near field (the field and its derivative from one
staging of the sources) against the two-pass form, which launch shapes with
two lane subgroups take: FP64 sums differ by rounding only, far below the
1e-12 parity bar; in mixed precision the 1e-6 bar (the truncation of the order
is the same in both).
Leaf sizes around the targets per lane (1, 2, 4), split lists, and shallow
problems whose L2P is a kernel of its own."""
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


@pytest.mark.parametrize("n,L,p", [(300, 5, 8), (2000, 5, 16), (4097, 4, 17), (9000, 1, 5), (1003, 2, 12), (5000, 3, 40)])
def test_one_pass_matches_two_passes(F, n, L, p):
    z, m, _ = W.uniform(n, seed=n)
    tree, md = F.build_tree(dev(z), L), dev(m)
    one = [host(x) for x in F.evaluate_field(F.plan(tree, p, 0.5, "fp64"), md)]
    two = [host(x) for x in F.evaluate_field(F.plan(tree, p, 0.5, "fp64", p2p_split=2, p2p_targets=4), md)]
    assert e2(one[0], two[0]) <= 1e-12 and e2(one[1], two[1]) <= 1e-12
    np.testing.assert_array_equal(one[0], host(F.evaluate(F.plan(tree, p, 0.5, "fp64"), md)))
    one = host(F.evaluate_field(F.plan(tree, p, 0.5, "mixed"), md)[1])
    two = host(F.evaluate_field(F.plan(tree, p, 0.5, "mixed", p2p_split=2, p2p_targets=4), md)[1])
    assert e2(one, two) <= 1e-6


def test_split_lists(F, orc):
    rng = np.random.default_rng(6)
    z = np.concatenate([1e-4 * (rng.random(6000) + 1j * rng.random(6000)), rng.random(2000) + 1j * rng.random(2000)])
    m = rng.standard_normal(z.size) + 1j * rng.standard_normal(z.size)
    tree, md = F.build_tree(dev(z), 3), dev(m)
    pl = F.plan(tree, 30, 0.5, "fp64")
    phi, dphi = F.evaluate_field(pl, md)
    assert e2(host(phi), orc.direct(z, m)) <= 1e-12
    assert e2(host(dphi), orc.direct_deriv_points(z, m, z)) <= 1e-12
    np.testing.assert_array_equal(host(phi), host(F.evaluate(pl, md)))
