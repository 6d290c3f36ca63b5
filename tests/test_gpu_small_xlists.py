"""X lists of small systems at p = 2, where P2L runs on the caller's stream up to
1,024 points and beside the upward pass above: evaluations, repeated, and the
adjoint against the oracle's sweep at FP32's bound, on points half of which lie
in a small cube."""
import numpy as np
import pytest

import workloads
from oracle import kifmm
from _parity import check

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ROOT = ((0.0, 0.0, 0.0), 1.0)


@pytest.mark.parametrize("profile", [False, True])
@pytest.mark.parametrize("n,leaf", [(100, 12), (300, 16), (1024, 16), (1025, 16)])
def test_small_x_lists(n, leaf, profile):
    from paper_2512_09478_amd import Plan
    print(f"small X lists n={n} leaf={leaf} profile={profile}", flush=True)
    rng = np.random.default_rng(n)
    x = rng.random((n, 3))
    x[n // 2:] = 0.3 + 0.02 * x[n // 2:]
    x = workloads.round_f32(x)
    q, gu = workloads.round_f32(rng.standard_normal(n)), workloads.round_f32(rng.standard_normal(n))
    gE = workloads.round_f32(rng.standard_normal((n, 3)))
    dev = lambda a: torch.tensor(a, dtype=torch.float32, device="cuda")
    G = Plan(torch.tensor(x, dtype=torch.float64, device="cuda"), "laplace", 2, leaf, root=ROOT, profile=profile)
    t, xl = G.tree(), G.list_csr("X")[0]
    size = np.asarray(t["end"]) - np.asarray(t["begin"])
    assert np.any((np.diff(np.asarray(xl)) > 0) & ~(np.asarray(t["is_leaf"]).astype(bool) & (size <= 8)))   # not summed directly
    O = kifmm.plan(x, "laplace", 2, leaf, True, 21, ROOT)
    uo, Eo = kifmm.forward(O, q)
    go, xo = kifmm.vjp(O, q, gu, gE)
    for _ in range(2):
        u, E = G.evaluate(dev(q))
        check("u", u, uo, 1e-5)
        check("E", E, Eo, 1e-5)
        gq, gx = G.backward(None, dev(gu), dev(gE))
        check("grad_charges", gq, go, 1e-5)
        check("grad_positions", gx, xo, 1e-5)
