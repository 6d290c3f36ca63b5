"""Upward and downward passes on wide levels: the forms of the translation
kernels that take two row blocks (above 1,024 non-leaves a level) and two column
blocks (above 4,096 boxes), at every surface size, with the exact and the
compressed M2L.

A small system, whose levels take the narrow forms, is compared with itself
inside a large one whose other points carry nothing: the same boxes and
densities, in launches of the wide forms, so that only rounding differs (the
M2L's partial sums are split otherwise, and the rounding of the check potentials
reaches the field amplified): 2e-5 for charges of both signs, 1e-4 at p >= 7."""
import numpy as np
import pytest

import workloads
from _parity import check

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SMALL, LARGE = 1200, 60000


@pytest.fixture(scope="module")
def points():
    rng = np.random.default_rng(41)
    return workloads.round_f32(0.49 * rng.random((SMALL, 3))), workloads.round_f32(0.51 + 0.48 * rng.random((LARGE, 3)))


def make(x, p, m2l_rtol):
    from paper_2512_09478_amd import Plan
    return Plan(torch.tensor(x, dtype=torch.float64, device="cuda"), "laplace", p, 2, root=((0.0, 0.0, 0.0), 1.0),
                m2l_rtol=m2l_rtol)


def widths(plan):
    """(non-leaves of each level, leaves)"""
    t = plan.tree()
    return np.bincount(t["level"][~t["is_leaf"]]), int(t["is_leaf"].sum())


def pad(a):
    a = np.asarray(a, np.float32)
    return torch.tensor(np.concatenate([a, np.zeros((LARGE,) + a.shape[1:], np.float32)]), device="cuda")


@pytest.mark.parametrize("m2l_rtol", [0.0, 1e-6])
@pytest.mark.parametrize("p", [2, 3, 4, 5, 6, 7, 8])
def test_wide_levels(points, p, m2l_rtol):
    print(f"wide levels p={p} m2l_rtol={m2l_rtol}", flush=True)
    x, far = points
    few, many = make(x, p, m2l_rtol), make(np.concatenate([x, far]), p, m2l_rtol)
    w, leaves = widths(few)
    assert w.max() <= 512 and leaves <= 4096
    w, leaves = widths(many)
    assert w.max() > 4096 and leaves > 32768 and np.any((w > 512) & (w < 4096))
    rng = np.random.default_rng(42)
    q, gu = rng.standard_normal(SMALL), rng.standard_normal(SMALL)
    gE, f = rng.standard_normal((SMALL, 3)), rng.standard_normal((SMALL, 3))
    dev = lambda a: torch.tensor(a, dtype=torch.float32, device="cuda")
    tol = 1e-4 if p >= 7 else 2e-5
    names = ("u", "E", "grad_charges", "grad_positions", "velocity")
    a = few.evaluate(dev(q)) + few.backward(dev(q), dev(gu), dev(gE)) + (few.evaluate_stokes(dev(f), 0.7),)
    b = many.evaluate(pad(q)) + many.backward(pad(q), pad(gu), pad(gE)) + (many.evaluate_stokes(pad(f), 0.7),)
    for name, s, l in zip(names, a, b):
        check(name, l[:SMALL], s.double().cpu().numpy(), tol)
