"""The FP64 logarithm of the near-field kernel: one leaf (N_levels 1), so the
result is the direct sum alone, against extended precision.

Distances whose squares sweep the table's 128 intervals, the edges of its
intervals, numbers just around 1, and the whole exponent range.  The bound: a
term q log r carries the rounding of r^2 (at most eps absolute in log r) and
two units in the last place of log r, the sum of n terms one rounding each,
at most eps * sqrt(n) * sum |q log r| for these random signs."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1311_1006_amd as F
    F.lib()
    return F


def distances(kind):
    if kind == "mantissas":
        return np.sqrt(0.75 + np.arange(1, 400) / 256.0)
    if kind == "edges":      # one unit around the interval edges of r^2
        e = np.concatenate([0.75 + np.arange(65) / 256.0, 1.0 + np.arange(65) / 128.0])
        return np.concatenate([np.sqrt(np.nextafter(e, 0)), np.sqrt(e), np.sqrt(np.nextafter(e, 2))])
    if kind == "one":
        return np.concatenate([1.0 + np.ldexp(1.0, -np.arange(1, 53)), 1.0 - np.ldexp(1.0, -np.arange(1, 53))])
    return np.ldexp(1.37, np.arange(-500, 500, 7))


@pytest.mark.parametrize("kind", ["mantissas", "edges", "one", "exponents"])
def test_direct_log_sum(F, kind):
    import torch
    d = distances(kind)
    z = np.concatenate([[0.0], d]) + 0j       # point 0 sees every distance
    q = np.random.default_rng(3).standard_normal(z.size)
    zd, qd = torch.from_numpy(z).cuda(), torch.from_numpy(q).cuda()
    u = F.evaluate_log(F.plan(F.build_tree(zd, 1), 4, 0.5, "fp64"), qd).cpu().numpy()
    r2 = d.astype(np.longdouble) ** 2 + np.finfo(np.float64).tiny     # the kernel's r^2
    lg = 0.5 * np.log(r2)
    ref = np.sum(q[1:].astype(np.longdouble) * lg)
    eps = np.finfo(np.float64).eps
    terms = np.abs(q[1:]) * (3 * np.abs(lg) + 1)
    bound = eps * float(np.sum(terms)) + eps * np.sqrt(d.size) * float(np.sum(np.abs(q[1:] * lg)))
    assert abs(float(u[0] - ref)) <= bound

