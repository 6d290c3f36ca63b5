"""Rounding of the near field: a target's largest terms, those of its own leaf,
are added last.

Every point of one leaf has a partner at distance 2^-6, whose field (4096 in
units of the charge, exact in FP32 but for the reciprocal root) is most of the
sum; some 30,000 terms of size 3, at distances of 0.1 and more, come from the
other seven leaves.  In a depth-1 tree all pairs are near, and eight lanes share
a target.  The lane with the
partner's term adds at most eight more after it, each rounded to half a unit in
the last place of a number below 8192: relative to 4096 sqrt(8) 2^-24 / sqrt(3) in
the root mean square, 1e-7; the far partial sums (of some 200, in 4,000 steps)
leave 7e-8, a unit in the last place of the reciprocal root, cubed, 1.8e-7: in
all below 5e-7.  With the partner first, the 4,000 terms after it leave
sqrt(4000) 2^-24 / sqrt(3) = 2.2e-6."""
import numpy as np
import pytest

import workloads
from oracle import direct
from _parity import rel

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

PAIRS, OTHERS = 32, 40000


def system():
    rng = np.random.default_rng(21)
    k = np.arange(2 * PAIRS)[::2]
    a = np.stack([k // 16, k // 4 % 4, (k + k // 4) % 4], 1) / 8 + 1 / 32
    x = np.concatenate([a, a + [1 / 64, 0, 0]]) + [0, 0.5, 0]   # octant 2 of the root
    y = workloads.round_f32(rng.random((OTHERS, 3)))
    y = y[(y[:, 0] >= 0.6) | (y[:, 1] < 0.4) | (y[:, 2] >= 0.6)]
    q = np.concatenate([np.ones(len(x)), workloads.round_f32(rng.standard_normal(len(y)))])
    return np.concatenate([x, y]), q, len(x)


@pytest.mark.parametrize("form", ["evaluate", "dipoles", "gradient", "clump"])
def test_own_leaf_last(form):
    from paper_2512_09478_amd import Plan
    print(f"near order {form}", flush=True)
    x, q, n = system()
    G = Plan(torch.tensor(x, dtype=torch.float64, device="cuda"), "laplace", 3, 64, True, 1, root=((0.0, 0.0, 0.0), 1.0))
    Q = torch.tensor(q, dtype=torch.float32, device="cuda")
    if form == "evaluate":
        E = G.evaluate(Q)[1]
    elif form == "dipoles":
        E = G.evaluate_dipoles(Q, torch.zeros((len(x), 3), device="cuda"))[1]
    elif form == "gradient":
        E = G.evaluate_gradient(Q)[1]
    else:   # clumps of one pebble: nothing but the self pair is left out
        off = torch.arange(len(x) + 1, device="cuda")
        G.set_clumps(off)
        E = G.clump_forces(Q, torch.tensor(x, device="cuda"), field=True)[2]
    _, ref, _ = direct.potential_field(x, q, targets=np.arange(n))
    err = rel(E[:n].cpu().numpy(), ref)
    print(f"    E of the pairs: {err:.2e}", flush=True)
    assert err < 5e-7
