"""tests/order_reference.py against the oracle: its field at the sources' leaves is the
oracle's FMM of the same order, and at a converged order its sums are the direct ones."""
import numpy as np
import pytest

from paper_1311_1006_amd import workloads as W
from order_reference import Order


def e2(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("n,L", [(64, 2), (700, 3), (1500, 4)])
def test_converged(orc, n, L):
    z, m, _ = W.uniform(n, seed=n)
    q = m.real + 0j
    ref = Order(orc, z, q, L, 0.5, 60)
    assert e2(ref.log(), orc.direct_log_points(z, q.real, z)) <= 1e-12
    y = W.uniform(200, seed=n + 1)[0]
    box = ref.leaf_of(y)
    y, box = y[box >= 0], box[box >= 0]
    assert y.size > 100
    phi, dphi = ref.points(y, box)
    assert e2(phi, orc.direct_points(z, q, y)) <= 1e-12
    assert e2(dphi, orc.direct_deriv_points(z, q, y)) <= 1e-10


@pytest.mark.parametrize("p", [1, 2, 5, 17])
def test_field_of_one_order(orc, p):
    # the derivative of the log's far field is the harmonic one: points a little off
    # the sources, the near field taken out on both sides
    n, L = 1500, 4
    z, m, _ = W.uniform(n, seed=3)
    ref = Order(orc, z, m, L, 0.5, p)
    _, _, far = orc.fmm(z, m, p, 0.5, L, parts=True)
    leaf = np.zeros(n, np.int64)
    lb = ref.base[L - 1]
    for g in range(4 ** (L - 1)):
        s, c = ref.range[lb + g]
        leaf[ref.perm[s:s + c]] = lb + g
    w = ((z - ref.c[leaf]) / ref.r[leaf])[:, None]
    mine = np.sum(ref.b[leaf] * w ** np.arange(p), axis=1)
    assert e2(mine, far) <= 1e-12
