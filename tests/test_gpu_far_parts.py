"""Leaf evaluation with items in parts of their targets.

A small system, whose items are divided, is compared with its own evaluation
inside a large one, whose items are whole: the same points and charges, and far
away enough uncharged points that there are more items than are divided.  Sums
of some hundred terms in another order differ by eps32 times the square root
of their number, below 1e-6; the two trees also split the M2L differently, and
the rounding of its check potentials reaches the field amplified, by at most
2e-5 in systems of both signs."""
import numpy as np
import pytest
import torch

from paper_2512_09478_amd import Plan

pytestmark = pytest.mark.gpu


def system(kind, n, seed):
    rng = np.random.default_rng(seed)
    if kind == "uniform":
        x = rng.random((n, 3))
    else:   # a dense clump in a thin cloud: leaves with long W lists
        x = np.concatenate([0.3 + 0.01 * rng.random((n // 2, 3)), rng.random((n - n // 2, 3))])
    return (0.49 * x).astype(np.float32).astype(np.float64)


@pytest.mark.parametrize("grad", [False, True])
@pytest.mark.parametrize("kind,n,leaf", [("uniform", 70, 16), ("uniform", 3000, 64), ("clump", 3000, 64),
                                         ("clump", 40000, 33)])
def test_parts(kind, n, leaf, grad):
    print(f"parts {kind} n={n} leaf={leaf} grad={grad}", flush=True)
    x = system(kind, n, n)
    rng = np.random.default_rng(1)
    far = (0.51 + 0.49 * rng.random((leaf * 9000, 3))).astype(np.float32).astype(np.float64)
    q = torch.from_numpy(rng.standard_normal(n).astype(np.float32)).cuda()
    root = ((0.0, 0.0, 0.0), 1.0)
    few = Plan(torch.from_numpy(x).cuda(), p=6, leaf_size=leaf, root=root)
    many = Plan(torch.from_numpy(np.concatenate([x, far])).cuda(), p=6, leaf_size=leaf, root=root)
    qm = torch.cat([q, torch.zeros(len(far), device="cuda")])
    if grad:
        a, b = few.evaluate_gradient(q), many.evaluate_gradient(qm)
    else:
        a, b = few.evaluate(q), many.evaluate(qm)
    for name, u, v in zip(("u", "E", "dE"), a, b):
        v = v[:n]
        err = ((u - v).double().norm() / v.double().norm()).item()
        print(f"  {name}: {err:.1e}", flush=True)
        assert torch.isfinite(u).all() and err < 2e-5
