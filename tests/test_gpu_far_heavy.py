"""Leaf evaluation of 512 to 1,024 work items whose heaviest leaves (the coarse
ones beside a dense clump, with long W lists) come late in leaf
order, past the 256 items that are divided most.  The FP32 path's bound."""
import numpy as np
import pytest

import workloads
from oracle import kifmm
from _parity import check

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ROOT = ((0.0, 0.0, 0.0), 1.0)


@pytest.mark.parametrize("n,m,leaf,width", [(16000, 4000, 32, 0.01), (15000, 3500, 40, 0.004)])
def test_heavy_leaves_late(n, m, leaf, width):
    from paper_2512_09478_amd import Plan
    print(f"heavy leaves n={n} leaf={leaf}", flush=True)
    rng = np.random.default_rng(3)
    x = rng.random((n, 3))
    x[:m] = width * x[:m] + 0.9 - width / 2
    x = workloads.round_f32(x)
    q = workloads.round_f32(rng.standard_normal(n))
    G = Plan(torch.tensor(x, dtype=torch.float64, device="cuda"), "laplace", 4, leaf, root=ROOT)
    t = G.tree()
    lf = t["is_leaf"]
    count = (t["end"] - t["begin"])[lf]
    off, _ = G.list_csr("W")
    items = -(-count // 64)
    assert 512 <= items.sum() <= 1024
    w = np.repeat((off[1:] - off[:-1])[lf], items)
    assert w.argmax() >= 256 and w.max() > 50
    O = kifmm.plan(x, "laplace", 4, leaf, True, 21, ROOT)
    uo, Eo = kifmm.forward(O, q)
    u, E = G.evaluate(torch.tensor(q, dtype=torch.float32, device="cuda"))
    check("u", u, uo, 1e-5)
    check("E", E, Eo, 1e-5)
    ug, Eg, _ = G.evaluate_gradient(torch.tensor(q, dtype=torch.float32, device="cuda"))
    check("u beside the gradient", ug, uo, 1e-5)
    check("E beside the gradient", Eg, Eo, 1e-5)
