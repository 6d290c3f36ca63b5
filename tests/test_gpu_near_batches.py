"""GPU near field at the edges of its staging: numbers of targets and of
staged points around the batch, wave and item sizes, many runs per leaf, and
points of two leaves whose coordinates round to one.

On a tree of depth 1 every pair is a near pair, so the direct sum over the
FP32-rounded positions is the reference.  A sum of FP32 terms, each right to a
few units of 2^-24, is held to 64 units in relative L2 (4e-6), a gradient,
whose terms cancel more, to 160 (1e-5).
"""
import numpy as np
import pytest

import workloads
from oracle import direct, kifmm
from _parity import check

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24
ROOT = ((0.0, 0.0, 0.0), 1.0)


def plan(x, p=3, leaf=8, max_depth=1, **kw):
    from paper_2512_09478_amd import Plan
    return Plan(torch.tensor(x, dtype=torch.float64, device="cuda"), "laplace", p, leaf, True, max_depth, root=ROOT,
                **kw)


def dev(a):
    return torch.tensor(a, dtype=torch.float32, device="cuda")


# leaf = n: one leaf of n points (its own, tested pairs only); leaf = 8: up to
# eight leaves (tested and untested pairs in one batch, batches that end inside a leaf)
@pytest.mark.parametrize("one_leaf", [True, False])
@pytest.mark.parametrize("n", [2, 15, 16, 17, 63, 64, 65, 511, 512, 513, 768, 769, 1025, 5000])
def test_all_pairs_near(n, one_leaf):
    print(f"near field n={n} one_leaf={one_leaf}", flush=True)
    rng = np.random.default_rng(100 + n)
    x = workloads.uniform_cube(rng, n)
    q, gu = workloads.round_f32(rng.standard_normal(n)), workloads.round_f32(rng.standard_normal(n))
    gE, m = workloads.round_f32(rng.standard_normal((n, 3))), workloads.round_f32(rng.standard_normal((n, 3)))
    G = plan(x, leaf=n if one_leaf else 8)
    u, E = G.evaluate(dev(q))
    gq, gx = G.backward(None, dev(gu), dev(gE))
    ud, Ed, _ = direct.potential_field(x, q)
    gqd, gxd = direct.vjp(x, q, gu, gE)
    check("u", u, ud, 64 * EPS)
    check("E", E, Ed, 64 * EPS)
    check("grad_charges", gq, gqd, 160 * EPS)
    check("grad_positions", gx, gxd, 160 * EPS)
    uq, Eq, Gq = G.evaluate_gradient(dev(q), dev(m))
    um, Em, Gm = direct.dipole_potential_field(x, q, m, grad=True)
    check("u of dipoles", uq, um, 160 * EPS)
    check("E of dipoles", Eq, Em, 160 * EPS)
    check("gradient of dipoles", Gq, Gm, 160 * EPS)


def test_leaves_that_meet_in_one_rounded_point():
    """0.5 -+ 2^-40 lie in different leaves and round to the same FP32 value:
    pairs of them are at distance zero and skipped, in whole items of such
    points and beside others."""
    print("points that straddle a face", flush=True)
    rng = np.random.default_rng(3)
    n = 200
    x = workloads.uniform_cube(rng, n)
    x[:80, 0] = 0.5 - 2.0 ** -40
    x[80:160] = x[:80]
    x[80:160, 0] = 0.5 + 2.0 ** -40
    q = workloads.round_f32(rng.standard_normal(n))
    f = workloads.round_f32(rng.standard_normal((n, 3)))
    G = plan(x)
    xr = workloads.round_f32(x)
    ud, Ed, _ = direct.potential_field(xr, q)
    u, E = G.evaluate(dev(q))
    check("u", u, ud, 64 * EPS)
    check("E", E, Ed, 64 * EPS)
    gq, gx = G.backward(None, dev(q), dev(f))
    gqd, gxd = direct.vjp(xr, q, q, f)
    check("grad_charges", gq, gqd, 160 * EPS)
    check("grad_positions", gx, gxd, 160 * EPS)


def test_leaf_with_many_runs():
    """A coarse leaf beside a dense face has far more near boxes than the 64
    runs a wave holds at once."""
    print("many runs", flush=True)
    rng = np.random.default_rng(4)
    x = workloads.uniform_cube(rng, 6000)
    x[:5900, 0] = 0.5 + 0.02 * x[:5900, 0]
    x[5900:, 0] *= 0.5
    x = workloads.round_f32(x)
    q = workloads.round_f32(rng.standard_normal(6000))
    G = plan(x, p=4, leaf=4, max_depth=21)
    off, _ = G.list_csr("N")
    assert np.max(off[1:] - off[:-1]) > 200
    u, E = G.evaluate(dev(q))
    O = kifmm.plan(x, "laplace", 4, 4, True, 21, ROOT)
    uo, Eo = kifmm.forward(O, q)
    check("u", u, uo, 1e-5)
    check("E", E, Eo, 1e-5)
