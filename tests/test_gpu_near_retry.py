"""Points of two leaves whose coordinates round to one, in every form of the near
field: 0.5 -+ 2^-40 lie in different leaves and are one FP32 value.  Pairs
between leaves run without a test for distance zero, so the items that hold such
a pair come out infinite or NaN and are done again with every pair tested.

On a tree of depth 1 every pair is near, and the direct sum over the rounded
positions, which leaves out pairs at distance zero, is the reference: sums of
FP32 terms to 64 units of 2^-24 in relative L2, those whose terms cancel more
(gradients, dipoles, the adjoint) to 160."""
import numpy as np
import pytest

import workloads
from oracle import clump, direct, stokes
from _parity import check

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24
N, HALF = 200, 80


@pytest.fixture(scope="module")
def system():
    rng = np.random.default_rng(31)
    x = workloads.uniform_cube(rng, N)
    x[:HALF, 0] = 0.5 - 2.0 ** -40
    x[HALF:2 * HALF] = x[:HALF]
    x[HALF:2 * HALF, 0] = 0.5 + 2.0 ** -40
    q = workloads.round_f32(rng.standard_normal(N))
    return x, workloads.round_f32(x), q, workloads.round_f32(rng.standard_normal((N, 3)))


def plan(x):
    from paper_2512_09478_amd import Plan
    G = Plan(torch.tensor(x, dtype=torch.float64, device="cuda"), "laplace", 3, 8, True, 1, root=((0.0, 0.0, 0.0), 1.0))
    t = G.tree()
    at = np.empty(N, int)
    at[t["perm"]] = np.searchsorted(t["end"][1:], np.arange(N), side="right")   # leaf of each point (level 1, key order)
    assert np.all(at[:HALF] != at[HALF:2 * HALF])
    return G


def dev(a):
    return torch.tensor(a, dtype=torch.float32, device="cuda")


def test_dipoles_and_gradient(system):
    print("straddling points: dipoles, gradient", flush=True)
    x, xr, q, m = system
    G = plan(x)
    ud, Ed, Gd = direct.dipole_potential_field(xr, q, m, grad=True)
    u, E = G.evaluate_dipoles(dev(q), dev(m))
    check("u of dipoles", u, ud, 160 * EPS)
    check("E of dipoles", E, Ed, 160 * EPS)
    u, E, D = G.evaluate_gradient(dev(q), dev(m))
    check("u of dipoles, gradient call", u, ud, 160 * EPS)
    check("E of dipoles, gradient call", E, Ed, 160 * EPS)
    check("gradient of dipoles", D, Gd, 160 * EPS)
    ud, Ed, Gd = direct.dipole_potential_field(xr, q, np.zeros((N, 3)), grad=True)
    u, E, D = G.evaluate_gradient(dev(q))
    check("u, gradient call", u, ud, 64 * EPS)
    check("E, gradient call", E, Ed, 64 * EPS)
    check("gradient", D, Gd, 160 * EPS)


def test_stokes(system):
    print("straddling points: Stokes", flush=True)
    x, xr, _, f = system
    u, p = plan(x).evaluate_stokes(dev(f), 0.7, pressure=True)
    check("velocity", u, stokes.direct(xr, f, 0.7), 64 * EPS)
    check("pressure", p, stokes.pressure_direct(xr, f), 160 * EPS)


def test_clumps(system):
    print("straddling points: clump forces and gradients", flush=True)
    x, xr, q, _ = system
    off = np.arange(0, N + 1, 4)
    rng = np.random.default_rng(32)
    cen = np.array([xr[a:b].mean(0) for a, b in zip(off[:-1], off[1:])])
    gF, gT = rng.standard_normal((len(off) - 1, 3)), rng.standard_normal((len(off) - 1, 3))
    G = plan(x)
    G.set_clumps(torch.tensor(off, device="cuda"))
    C = torch.tensor(cen, device="cuda")
    F, T, E = G.clump_forces(dev(q), C, field=True)
    _, full, _ = direct.potential_field(xr, q)
    own = np.concatenate([direct.potential_field(xr[a:b], q[a:b])[1] for a, b in zip(off[:-1], off[1:])])
    check("E without the clump's own", E, full - own, 64 * EPS)
    Fo, To = clump.clump_reduce(xr, q, full - own, off, cen)
    check("force", F, Fo, 160 * EPS)
    check("torque", T, To, 160 * EPS)
    gq, gx, gX = G.clump_forces_backward(dev(q), C, torch.tensor(gF, device="cuda"), torch.tensor(gT, device="cuda"))
    qd, Eb, xd, Xd = clump.clump_vjp(xr, q, full, off, cen, gF, gT)
    qf, xf = direct.vjp(xr, q, np.zeros(N), Eb)
    check("dL/dq", gq, qd + qf, 160 * EPS)
    check("dL/dx", gx, xd + xf, 160 * EPS)
    check("dL/dX", gX, Xd, 160 * EPS)
