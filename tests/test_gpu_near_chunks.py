"""Near-field units taken from the counter one, two and four at a time: thin
sheets of small leaves, from about one leaf a resident block (1,024 of them) to
ten, odd counts whose last chunk runs past the units, repeated calls (the counter
starts again at zero) and the adjoint.  Against the oracle's sweep at FP32's
bound."""
import numpy as np
import pytest

import workloads
from oracle import kifmm
from _parity import check

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ROOT = ((0.0, 0.0, 0.0), 1.0)


@pytest.mark.parametrize("n,leaf", [(2500, 4), (9001, 4), (30011, 4), (30000, 6)])
def test_light_units(n, leaf):
    from paper_2512_09478_amd import Plan
    print(f"light units n={n} leaf={leaf}", flush=True)
    rng = np.random.default_rng(n)
    x = rng.random((n, 3))
    x[:, 2] = 0.3 + 1e-3 * x[:, 2]
    x = workloads.round_f32(x)
    q, gu = workloads.round_f32(rng.standard_normal(n)), workloads.round_f32(rng.standard_normal(n))
    gE = workloads.round_f32(rng.standard_normal((n, 3)))
    dev = lambda a: torch.tensor(a, dtype=torch.float32, device="cuda")
    G = Plan(torch.tensor(x, dtype=torch.float64, device="cuda"), "laplace", 4, leaf, root=ROOT)
    O = kifmm.plan(x, "laplace", 4, leaf, True, 21, ROOT)
    idx = np.sort(rng.choice(n, 500, replace=False))
    uo, Eo = kifmm.forward(O, q, targets=idx)
    for _ in range(2):
        u, E = G.evaluate(dev(q))
        check("u", u[idx], uo, 1e-5)
        check("E", E[idx], Eo, 1e-5)
    gq, gx = G.backward(None, dev(gu), dev(gE))
    go, xo = kifmm.vjp(O, q, gu, gE, targets=idx)
    check("grad_charges", gq[idx], go, 1e-5)
    check("grad_positions", gx[idx], xo, 1e-5)
