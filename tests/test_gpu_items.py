"""More work items than the merge sort takes (65,536), ordered by one pass over
their keys: every target is in one item, so the sums of a tree of tiny leaves are
those of a tree of large ones up to the method's error (p = 6, charges of one
sign: below 1e-5 of the potential)."""
import numpy as np
import pytest

import workloads
from _parity import check

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [150000, 250007])
def test_many_items(n):
    from paper_2512_09478_amd import Plan
    print(f"many items n={n}", flush=True)
    rng = np.random.default_rng(n)
    x = torch.tensor(workloads.round_f32(rng.random((n, 3))), device="cuda")
    q = torch.tensor(0.5 + rng.random(n), dtype=torch.float32, device="cuda")
    root = ((0.0, 0.0, 0.0), 1.0)
    many, few = Plan(x, p=6, leaf_size=2, root=root), Plan(x, p=6, leaf_size=128, root=root)
    assert many.counts()["leaves"] > 65536 > few.counts()["leaves"]
    for p in (many, few):
        p.rebuild(x)
    u, _ = many.evaluate(q)
    v, _ = few.evaluate(q)
    check("u", u, v.double().cpu().numpy(), 2e-5)
    g, _ = many.backward(None, q, torch.zeros((n, 3), device="cuda"))
    check("grad_charges", g, v.double().cpu().numpy(), 2e-5)
