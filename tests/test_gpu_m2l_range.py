"""The FP32 path's M2L by bf16 pieces over FP32's range, and on one-signed charges.

Charges times 2^-116 (about 1e-35) leave densities whose second and third
pieces are below the smallest normal number unless they are scaled; FP32
instructions held them to their last places but for subnormal terms 2^-33 of
the largest.  So the sums of tiny charges, divided by the factor, may be no
further from the oracle than those of the charges themselves but for another
draw of the same rounding: half as much again.  Without the scaling they were
two to five times as far.

One-signed charges (the same sums as gravity, up to a constant) take the same
products: FP32's bound."""
import numpy as np
import pytest

import workloads
from oracle import kifmm
from _parity import check, rel

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TINY = 2.0 ** -116
ROOT = ((0.0, 0.0, 0.0), 1.0)


def plan(x, p, leaf, m2l_rtol):
    from paper_2512_09478_amd import Plan
    return Plan(torch.tensor(x, dtype=torch.float64, device="cuda"), "laplace", p, leaf, root=ROOT, m2l_rtol=m2l_rtol)


def dev(a):
    return torch.tensor(a, dtype=torch.float32, device="cuda")


def points(kind, n):
    rng = np.random.default_rng(n)
    x = rng.random((n, 3))
    if kind == "clump":   # a dense clump in a thin cloud: X lists beside the V lists
        x[: n // 2] = 0.3 + 0.01 * x[: n // 2]
    return workloads.round_f32(x), rng


@pytest.mark.parametrize("m2l_rtol", [0.0, 1e-6])
@pytest.mark.parametrize("kind,n,p,leaf", [("uniform", 20000, 4, 64), ("uniform", 12000, 6, 64), ("clump", 8000, 6, 16),
                                           ("clump", 6000, 3, 40)])
def test_tiny_charges(kind, n, p, leaf, m2l_rtol):
    print(f"tiny charges {kind} n={n} p={p} m2l_rtol={m2l_rtol}", flush=True)
    x, rng = points(kind, n)
    q, gu = workloads.round_f32(rng.standard_normal(n)), workloads.round_f32(rng.standard_normal(n))
    gE = workloads.round_f32(rng.standard_normal((n, 3)))
    O = kifmm.plan(x, "laplace", p, leaf, True, 21, ROOT, m2l_rtol=m2l_rtol)
    uo, Eo = kifmm.forward(O, q)
    G = plan(x, p, leaf, m2l_rtol)
    u, E = [a.double().cpu().numpy() for a in G.evaluate(dev(q))]
    ut, Et = [a.double().cpu().numpy() / TINY for a in G.evaluate(dev(q * TINY))]
    print(f"    u {rel(u, uo):.2e} tiny {rel(ut, uo):.2e}   E {rel(E, Eo):.2e} tiny {rel(Et, Eo):.2e}", flush=True)
    assert rel(ut, uo) <= 1.5 * rel(u, uo) and rel(Et, Eo) <= 1.5 * rel(E, Eo)
    # both right-hand sides in one launch, one of them tiny: its share of the gradient
    # scales, the other's stays as it is
    gq, gx = G.backward(dev(q), dev(gu), dev(gE))
    gqt, gxt = G.backward(dev(q * TINY), dev(gu), dev(gE))
    assert torch.equal(gq, gqt)
    check("grad_positions", gxt.double() / TINY, gx.double().cpu().numpy(), 2e-6)
    assert not any(bool(a.any()) for a in G.evaluate(torch.zeros(n, device="cuda")))


@pytest.mark.parametrize("p,m2l_rtol", [(4, 0.0), (5, 0.0), (6, 0.0), (6, 1e-6)])
def test_one_signed_charges(p, m2l_rtol):
    """FP32's own distance from the oracle here, measured with FP32 instructions
    at 20,000 to 120,000 points: u to 3e-7, E to 1.8e-5, where E is the small
    difference of the far field's large terms."""
    n = 20000
    print(f"one-signed charges p={p} m2l_rtol={m2l_rtol}", flush=True)
    x, rng = points("uniform", n)
    q = workloads.round_f32(0.5 + rng.random(n))
    O = kifmm.plan(x, "laplace", p, 64, True, 21, ROOT, m2l_rtol=m2l_rtol)
    uo, Eo = kifmm.forward(O, q)
    u, E = plan(x, p, 64, m2l_rtol).evaluate(dev(q))
    check("u", u, uo, 1e-6)
    check("E", E, Eo, 2e-5)
