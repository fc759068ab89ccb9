"""Expansion orders whose coefficient rows are a multiple of 64 bytes (they are
stored with one coefficient of padding) and their neighbours, in both precisions,
through every reader of the rows: evaluation, field, evaluation at other points, the
adjoint and the fixed-memory evaluation, against the oracle's FMM of the same
order (parity: 1e-12; mixed: FP32 rounding, 1e-6 against the same order in FP64)."""
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


@pytest.mark.parametrize("n,L", [(900, 2), (9000, 5)])
@pytest.mark.parametrize("p", [7, 8, 9, 12, 15, 16, 17, 20, 24])
def test_rows_in_every_reader(orc, F, n, L, p):
    z, m, _ = W.uniform(n, seed=p)
    tree, md = F.build_tree(dev(z), L), dev(m)
    ref = orc.fmm(z, m, p, 0.5, L)
    pl = F.plan(tree, p, 0.5, "fp64")
    phi = host(F.evaluate(pl, md))
    assert e2(phi, ref) <= 1e-12
    phi2, dphi = F.evaluate_field(pl, md)
    assert e2(host(phi2), ref) <= 1e-12
    pm = F.plan(tree, p, 0.5, "mixed")
    assert e2(host(F.evaluate(pm, md)), phi) <= 1e-6
    assert e2(host(F.evaluate_field(pm, md)[1]), host(dphi)) <= 1e-5
    # other points: the sources' own positions, a little beside
    y = dev(z[:200] + 1e-9)
    ya, yb = F.evaluate_points(pl, md, y), F.evaluate_points(pm, md, y)
    assert e2(host(yb), host(ya)) <= 1e-6
    out = dev(np.zeros(n, np.complex128))
    F.evaluate_static(pl, md, out)
    assert np.array_equal(host(out), phi)
    # transposed: <g, F m> = <F^T g, m> with F^T g read off the adjoint
    g = np.random.default_rng(p).standard_normal(n) + 1j * np.random.default_rng(p + 1).standard_normal(n)
    F.evaluate(pl, md)
    gm, _ = F.evaluate_adjoint(pl, md, dev(g))
    lhs, rhs = np.vdot(g, phi), np.vdot(host(gm), m)
    assert abs(lhs.real - rhs.real) <= 1e-12 * np.linalg.norm(g) * np.linalg.norm(phi)


def test_fixed_memory_limit_leaves_out_the_padding(F):
    # 66.8 MB of 67.1 MB without the rows' padding, 68.2 MB with it
    n, L = 1390000, 9
    z, m, _ = W.uniform(n, seed=1)
    pl = F.plan(F.build_tree(dev(z), L), 16, 0.5, "mixed")
    md = dev(m)
    phi = host(F.evaluate(pl, md))
    assert pl.stats()["static_bytes"] <= 64 << 20
    out = dev(np.zeros(n, np.complex128))
    F.evaluate_static(pl, md, out)
    assert np.array_equal(host(out), phi)


@pytest.mark.parametrize("p", [1, 3, 4, 5, 8, 9, 12, 13, 17, 20, 21, 24, 25, 28, 29, 32])
def test_m2l_steps_by_order(orc, F, p):
    # every count of matrix steps of the automatic shape, around its edges: the
    # oracle's FMM of the same order
    z, m, _ = W.uniform(9000, seed=p)
    pl = F.plan(F.build_tree(dev(z), 5), p, 0.5, "fp64")
    assert e2(host(F.evaluate(pl, dev(m))), orc.fmm(z, m, p, 0.5, 5)) <= 1e-12


@pytest.mark.parametrize("p", [33, 36, 37, 40, 41, 44, 45, 48, 49, 52, 53, 56, 57, 60, 61, 64])
@pytest.mark.parametrize("n,L", [(3000, 3), (9000, 5)])
def test_m2l_steps_of_high_orders(orc, F, p, n, L):
    # converged: the direct sum, to the parity bar
    z, m, _ = W.uniform(n, seed=p)
    ref, md, tree = orc.direct(z, m), dev(m), F.build_tree(dev(z), L)
    assert e2(host(F.evaluate(F.plan(tree, p, 0.5, "fp64"), md)), ref) <= 1e-12
    assert e2(host(F.evaluate(F.plan(tree, p, 0.5, "mixed"), md)), ref) <= 1e-6
