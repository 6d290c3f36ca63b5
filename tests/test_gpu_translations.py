"""GPU upward and downward passes at every surface size, with the exact and
the compressed M2L, on levels of one box, of partial groups of 16 boxes and of
more boxes than one block takes."""
import numpy as np
import pytest

import workloads
from oracle import kifmm
from _parity import check

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# n points, leaf: up to 740 non-leaf boxes in the widest level (p = 2, 9000 points)
@pytest.mark.parametrize("p,n,leaf", [(2, 300, 8), (2, 9000, 2), (3, 3000, 6), (4, 9000, 2), (5, 3000, 6), (6, 300, 4),
                                      (6, 9000, 3), (7, 2000, 6), (8, 2500, 6)])
@pytest.mark.parametrize("m2l_rtol", [0.0, 1e-6])
def test_sweep_parity(p, n, leaf, m2l_rtol):
    from paper_2512_09478_amd import Plan
    print(f"sweep p={p} n={n} leaf={leaf} m2l_rtol={m2l_rtol}", flush=True)
    w = workloads.make(2, n=n, seed=50 + p)
    G = Plan(torch.tensor(w.positions, dtype=torch.float64, device="cuda"), w.kernel, p, leaf, root=w.root,
             m2l_rtol=m2l_rtol)
    u, E = G.evaluate(torch.tensor(w.charges, dtype=torch.float32, device="cuda"))
    O = kifmm.plan(w.positions, w.kernel, p, leaf, True, 21, w.root, m2l_rtol=m2l_rtol)
    uo, Eo = kifmm.forward(O, w.charges)
    # 1e-4 at p = 8, where FP32 rounding of the equivalent densities limits the field
    tol = 1e-4 if p >= 7 else 1e-5
    check("u", u, uo, tol)
    check("E", E, Eo, tol)
