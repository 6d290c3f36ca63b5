"""The sums whose speed is followed, through the calls a user's program makes.

A case names a particle set, the plan's options and one use of the plan:

  evaluate   potential and field of charges on a fixed plan
  fit        the same, then the gradients of a loss on them (charges, positions)
  step       two time steps of moving particles: re-tree, potential and field
  train      the same two steps, each with the gradients as well
  clump      force and torque of registered rigid clumps, and their gradients
  dipoles    potential and field of charges with point dipoles
  gradient   the same with the field gradient
  stokes     velocity and pressure of point forces

The particle sets are those of the repository's workloads (uniform cube,
clustered charges, rigid clumps, Plummer sphere, periodic platelets), drawn on
the GPU.  A time step moves every particle by N(0, drift^2) per axis.
"""
import math

import numpy as np
import torch

from paper_2512_09478_amd import Plan

VISCOSITY = 0.7
#: all-pairs sums in 64 bits stay in seconds up to this many points
EXACT_POINTS = 131_072

BASE = dict(kernel="laplace", p=6, leaf=128, adaptive=True, precision="split_bf16", m2l_rtol=1e-6, drift=0.0)


def _case(**kw):
    return {**BASE, **kw}


def listed():
    return [
        # one small system evaluated over and over on its plan: launches and latency
        _case(name="evaluate_uniform_4096", use="evaluate", points="uniform", n=4096, p=4, leaf=64, adaptive=False,
              precision="fp32", m2l_rtol=0.0),
        # a small particle simulation: every step re-builds the tree
        _case(name="step_clustered_10k", use="step", points="clustered", n=10_000, drift=1e-5),
        # a medium one whose particles cross cells from step to step, odd count
        _case(name="step_clustered_100k", use="step", points="clustered", n=100_003, drift=1e-3),
        # a plan with the library's defaults (FP32, exact operators), odd count
        _case(name="evaluate_clustered_131k_fp32", use="evaluate", points="clustered", n=131_071, precision="fp32",
              m2l_rtol=0.0),
        # a periodic cell of platelets, in time steps
        _case(name="step_platelets_55k", use="step", points="platelets", n=54_700, leaf=64, precision="fp32",
              m2l_rtol=0.0, drift=1e-5),
        # rigid clumps of eight pebbles: the force law of a granular simulation and its gradients
        _case(name="clump_200k", use="clump", points="clumps", n=200_000),
        # charges with dipoles, up to the field gradient (forces on dipole grains), odd count
        _case(name="gradient_clustered_262k", use="gradient", points="clustered", n=262_147),
        # charges fitted to a field: evaluation and gradients on one plan
        _case(name="fit_uniform_524k", use="fit", points="uniform", n=524_288),
        # the benchmark's workload on its FP32 path
        _case(name="evaluate_clustered_1M_fp32", use="evaluate", points="clustered", n=1_048_576, precision="fp32"),
        # the benchmark's step: re-tree, forward and adjoint
        _case(name="train_clustered_1M", use="train", points="clustered", n=1_048_576, drift=1e-5),
        # point forces in a viscous fluid, velocity and pressure
        _case(name="stokes_clustered_1M", use="stokes", points="clustered", n=1_048_576),
        # the largest: a self-gravitating sphere
        _case(name="evaluate_plummer_8M", use="evaluate", points="plummer", n=8_388_608, kernel="gravity", p=8,
              leaf=256),
    ]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    use = rng.choice(["evaluate", "evaluate", "fit", "step", "train", "clump", "dipoles", "gradient", "stokes"])
    if use == "clump":
        points, n = "clumps", 8 * _size(rng, 500, 60_000)
    elif use in ("step", "evaluate") and rng.random() < 0.25:
        points, n = "platelets", 1094 * rng.randint(4, 50)
    elif use in ("evaluate", "fit", "train") and rng.random() < 0.3:
        points, n = "plummer", _size(rng, 20_000, 2_000_000)
    else:
        points, n = rng.choice(["uniform", "clustered"]), _size(rng, 1_000, 1_000_000)
    c = _case(use=use, points=points, n=n, p=rng.choice([4, 6, 6, 6]), leaf=rng.choice([64, 128, 128]),
              precision=rng.choice(["split_bf16", "fp32"]), m2l_rtol=rng.choice([1e-6, 1e-6, 0.0]))
    if points == "plummer":
        c.update(kernel="gravity", p=rng.choice([6, 8]), leaf=rng.choice([128, 256]))
    if points == "platelets":
        c.update(leaf=64)
    if use in ("step", "train"):
        c.update(drift=rng.choice([1e-5, 1e-3]))
    return c


# ---------------------------------------------------------------- inputs
def _f32(x):
    return x.to(torch.float32).to(torch.float64)


def _inside(x):
    return x.clamp_(0.0, float(np.nextafter(np.float32(1.0), np.float32(0.0))))


def _uniform(g, n):
    return _inside(_f32(torch.rand((n, 3), generator=g, device="cuda", dtype=torch.float64)))


def _clustered(g, n):
    """60 % uniform, 40 % in 20 Gaussian clusters of width 0.02, tails folded back into the cube."""
    nu = int(round(0.6 * n))
    xu = torch.rand((nu, 3), generator=g, device="cuda", dtype=torch.float64)
    cen = torch.rand((20, 3), generator=g, device="cuda", dtype=torch.float64)
    which = torch.randint(0, 20, (n - nu,), generator=g, device="cuda")
    xc = cen[which] + 0.02 * torch.randn((n - nu, 3), generator=g, device="cuda", dtype=torch.float64)
    return _inside(_f32(torch.cat([xu, 1.0 - (1.0 - xc.abs()).abs()])))


def _plummer(g, n):
    """A Plummer sphere of scale 0.1 truncated at radius 1."""
    top = (1.0 + 0.1 ** 2) ** -1.5   # mass fraction inside the truncation radius
    u = (torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * top).clamp_min_(1e-12)
    r = 0.1 / torch.sqrt(u ** (-2.0 / 3.0) - 1.0)
    d = torch.randn((n, 3), generator=g, device="cuda", dtype=torch.float64)
    return _f32(d / d.norm(dim=1, keepdim=True) * r[:, None])


def _clumps(g, count):
    """Clumps of eight pebbles (cube corners, edge 0.6 R), randomly turned, in a shuffled set of
    lattice cells with the bounding spheres filling 30 % of a cell and jittered inside it."""
    side = max(1, math.ceil(count ** (1.0 / 3.0) - 1e-9))
    cell = 1.0 / side
    R = cell * (0.3 * 0.75 / math.pi) ** (1.0 / 3.0)
    at = torch.randperm(side ** 3, generator=g, device="cuda")[:count]
    ijk = torch.stack([at // (side * side), (at // side) % side, at % side], dim=1).to(torch.float64)
    jit = torch.rand((count, 3), generator=g, device="cuda", dtype=torch.float64) * (cell - 2 * R) + R
    cen = _f32(ijk * cell + jit)
    q = torch.randn((count, 4), generator=g, device="cuda", dtype=torch.float64)
    w, x, y, z = (q / q.norm(dim=1, keepdim=True)).unbind(1)
    rot = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w),
                       2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w),
                       2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)], dim=1).view(-1, 3, 3)
    s = torch.tensor([-0.3, 0.3], device="cuda", dtype=torch.float64) * R
    corners = torch.cartesian_prod(s, s, s)
    pts = cen[:, None, :] + (corners[None, :, None, :] * rot[:, None, :, :]).sum(-1)
    return _inside(_f32(pts.reshape(-1, 3))), cen


def _platelets(seed, count, rings=14, a=0.01):
    """Two-layer hexagonal platelets of 2 x 547 pebbles, +1 and -1, without overlap in the periodic cell."""
    rng = np.random.default_rng(seed)
    m = rings - 1
    lay = np.array([(a * (i + 0.5 * j), a * math.sqrt(0.75) * j, 0.0)
                    for i in range(-m, m + 1) for j in range(-m, m + 1) if abs(i + j) <= m])
    one = np.concatenate([lay, lay + np.array([0.5 * a, a / math.sqrt(12.0), a * math.sqrt(2.0 / 3.0)])])
    cen = []
    while len(cen) < count:
        c = rng.random(3)
        d = np.abs((np.array(cen).reshape(-1, 3) - c + 0.5) % 1.0 - 0.5)
        if not np.any((np.hypot(d[:, 0], d[:, 1]) < 2 * a * rings) & (d[:, 2] < 3 * a)):
            cen.append(c)
    x = (np.array(cen)[:, None, :] + one[None]).reshape(-1, 3) % 1.0
    x = x.astype(np.float32).astype(np.float64)
    x[x >= 1.0] = 0.0
    q = np.tile(np.repeat([1.0, -1.0], lay.shape[0]), count)
    return torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda().float()


def _inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    n, d = case["n"], {}
    randn = lambda *shape: torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)
    if case["points"] == "platelets":
        d["x"], d["q"] = _platelets(seed, n // 1094)
    elif case["points"] == "clumps":
        d["x"], d["centers"] = _clumps(g, n // 8)
        d["q"] = randn(n)
        d["offsets"] = torch.arange(0, n + 1, 8, device="cuda", dtype=torch.int64)
        d["gF"], d["gT"] = randn(n // 8, 3).double(), randn(n // 8, 3).double()
    else:
        d["x"] = {"uniform": _uniform, "clustered": _clustered, "plummer": _plummer}[case["points"]](g, n)
        q = randn(n)
        d["q"] = torch.ones_like(q) if case["points"] == "plummer" else q - q.mean()
    if case["use"] in ("fit", "train"):
        d["gu"], d["gE"] = randn(n), randn(n, 3)
    if case["use"] in ("dipoles", "gradient"):
        d["m"] = 0.01 * randn(n, 3)
    if case["use"] == "stokes":
        d["f"] = randn(n, 3)
    if case["use"] in ("step", "train"):
        y = d["x"] + case["drift"] * randn(n, 3).double()
        if case["points"] == "platelets":
            y = _f32(y % 1.0)
            y[y >= 1.0] = 0.0
        elif case["points"] == "plummer":
            y = _f32(y).clamp_(-1.0, 1.0)
        else:
            y = _inside(_f32(y))
        d["y"] = y.contiguous()
    return d


def prepare(case, seed):
    d = _inputs(case, seed)
    root = ((-1.0, -1.0, -1.0), 2.0) if case["points"] == "plummer" else ((0.0, 0.0, 0.0), 1.0)
    plan = Plan(d["x"], kernel=case["kernel"], p=case["p"], leaf_size=case["leaf"], adaptive=case["adaptive"],
                max_depth=12 if case["points"] == "plummer" else 21, precision=case["precision"], root=root,
                periodic=case["points"] == "platelets", m2l_rtol=case["m2l_rtol"])
    if case["use"] == "clump":
        plan.set_clumps(d["offsets"])
    return dict(d, case=case, plan=plan)


def run(state):
    plan, use = state["plan"], state["case"]["use"]
    if use == "evaluate":
        return plan.evaluate(state["q"])
    if use == "fit":
        u, E = plan.evaluate(state["q"])
        return (u, E, *plan.backward(None, state["gu"], state["gE"]))
    if use in ("step", "train"):
        out = []
        for x in (state["y"], state["x"]):
            plan.rebuild(x)
            out += plan.evaluate(state["q"])
            if use == "train":
                out += plan.backward(None, state["gu"], state["gE"])
        return out
    if use == "clump":
        F, T, E = plan.clump_forces(state["q"], state["centers"], field=True)
        gq, gx, gX = plan.clump_forces_backward(state["q"], state["centers"], state["gF"], state["gT"])
        # the 64-bit sums run over 32-bit fields and have their accuracy
        return F.float(), T.float(), E, gq, gx, gX.float()
    if use == "dipoles":
        return plan.evaluate_dipoles(state["q"], state["m"])
    if use == "gradient":
        return plan.evaluate_gradient(state["q"], state["m"])
    return plan.evaluate_stokes(state["f"], VISCOSITY, pressure=True)


# ---------------------------------------------------------------- necessary work
def work(case):
    """Inputs read once and outputs written once; operations of the method.

    A point has about 10 leaf sizes of near neighbours and about 850 / leaf
    far box pairs to its share (counted on these particle sets), of 2 k^2
    operations each with k the surface size 6 (p - 1)^2 + 2, or the rank that
    the truncated operators keep of it.
    """
    n, p, use = case["n"], case["p"], case["use"]
    k = 6 * (p - 1) ** 2 + 2
    if case["m2l_rtol"] > 0:
        k = {4: 56, 6: 116, 8: 124}.get(p, k)
    near, far = min(n, 10 * case["leaf"]), 2 * k * k * 850.0 / case["leaf"]
    # bytes a point in and out, operations a near pair, far sweeps, passes
    nbytes, pair, sweeps, times = {
        "evaluate": (20, 20, 1, 1),
        "fit": (56, 62, 2, 1),
        "step": (44, 20, 1, 2),
        "train": (80, 62, 2, 2),
        "clump": (50, 62, 2, 1),
        "dipoles": (32, 30, 1, 1),
        "gradient": (56, 45, 1, 1),
        "stokes": (28, 26, 4, 1),
    }[use]
    return {"bytes": float(times) * n * nbytes, "flops": times * n * (near * pair + far * sweeps)}


# ---------------------------------------------------------------- the sums themselves, in 64 bits
def _pairs(x, rows):
    """(dx, dy, dz, 1/r) from the points `rows` to all points; 1/r = 0 at distance zero."""
    d = [x[rows, k][:, None] - x[:, k][None, :] for k in range(3)]
    r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2]
    ri = torch.where(r2 > 0, r2, torch.ones_like(r2)).rsqrt_()
    return d, torch.where(r2 > 0, ri, torch.zeros_like(ri))


def _rows(n):
    step = max(1, 40_000_000 // n)
    return [slice(i, min(n, i + step)) for i in range(0, n, step)]


def _sum_charges(x, q, c, m=None, grad=False):
    u, E, G = [], [], []
    for rows in _rows(x.shape[0]):
        d, ri = _pairs(x, rows)
        r2, r3 = ri * ri, ri * ri * ri
        if m is None:
            u.append(ri @ q)
            E.append(torch.stack([(r3 * d[a]) @ q for a in range(3)], dim=1))
            continue
        mr = d[0] * m[:, 0] + d[1] * m[:, 1] + d[2] * m[:, 2]
        t = 3.0 * mr * r3 * r2
        g = q * r3 - t
        u.append((ri * q - mr * r3).sum(1))
        E.append(torch.stack([(g * d[a] + m[:, a] * r3).sum(1) for a in range(3)], dim=1))
        if grad:
            coef = 5.0 * t * r2 - 3.0 * q * r3 * r2
            w = 3.0 * r3 * r2
            G.append(torch.stack([(coef * d[a] * d[b] - w * (m[:, a] * d[b] + m[:, b] * d[a]) +
                                   (g if a == b else 0.0)).sum(1)
                                  for a, b in ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))], dim=1))
    out = [c * torch.cat(u), c * torch.cat(E)]
    return out + [c * torch.cat(G)] if grad else out


def _sum_adjoint(x, q, c, gu, gE):
    """d/dq and d/dx of sum gu u + gE . E."""
    psi, xb = [], []
    for rows in _rows(x.shape[0]):
        d, ri = _pairs(x, rows)
        r3 = ri * ri * ri
        rj = d[0] * gE[:, 0] + d[1] * gE[:, 1] + d[2] * gE[:, 2]
        psi.append((ri * gu - rj * r3).sum(1))
        rk = d[0] * gE[rows, 0][:, None] + d[1] * gE[rows, 1][:, None] + d[2] * gE[rows, 2][:, None]
        qk, uk = q[rows][:, None], gu[rows][:, None]
        g = -r3 * (uk * q + qk * gu) - 3.0 * r3 * ri * ri * (q * rk - qk * rj)
        xb.append(torch.stack([(g * d[a] + r3 * (q * gE[rows, a][:, None] - qk * gE[:, a])).sum(1)
                               for a in range(3)], dim=1))
    return [c * torch.cat(psi), c * torch.cat(xb)]


def exact(case, seed):
    use = case["use"]
    if case["n"] > EXACT_POINTS or case["points"] == "platelets":
        return None
    d = {k: v.double() if v.is_floating_point() else v for k, v in _inputs(case, seed).items()}
    c = -1.0 if case["kernel"] == "gravity" else 1.0 / (4.0 * math.pi)
    x, q = d["x"], d["q"]
    if use == "evaluate":
        return _sum_charges(x, q, c)
    if use == "fit":
        return _sum_charges(x, q, c) + _sum_adjoint(x, q, c, d["gu"], d["gE"])
    if use in ("step", "train"):
        out = []
        for pos in (d["y"], x):
            out += _sum_charges(pos, q, c)
            if use == "train":
                out += _sum_adjoint(pos, q, c, d["gu"], d["gE"])
        return out
    if use == "clump":
        E = _sum_charges(x, q, c)[1]
        r = x - d["centers"].repeat_interleave(8, dim=0)
        f = q[:, None] * E
        F, T = f.view(-1, 8, 3).sum(1), torch.linalg.cross(r, f).view(-1, 8, 3).sum(1)
        gF, gT = d["gF"].repeat_interleave(8, dim=0), d["gT"].repeat_interleave(8, dim=0)
        gq, gx = _sum_adjoint(x, q, c, torch.zeros_like(q), q[:, None] * (gF + torch.linalg.cross(gT, r)))
        own = q[:, None] * torch.linalg.cross(E, gT)
        gq = gq + (gF * E).sum(1) + (gT * torch.linalg.cross(r, E)).sum(1)
        # the pebble fields leave out the pairs inside a clump, which the sums do not show
        return F, T, None, gq, gx + own, -own.view(-1, 8, 3).sum(1)
    if use in ("dipoles", "gradient"):
        return _sum_charges(x, q, c, d["m"], use == "gradient")
    f, vel, prs = d["f"], [], []
    for rows in _rows(x.shape[0]):
        dd, ri = _pairs(x, rows)
        t = (dd[0] * f[:, 0] + dd[1] * f[:, 1] + dd[2] * f[:, 2]) * ri * ri * ri
        vel.append(torch.stack([(f[:, a] * ri + t * dd[a]).sum(1) for a in range(3)], dim=1))
        prs.append(t.sum(1))
    return [torch.cat(vel) / (8.0 * math.pi * VISCOSITY), torch.cat(prs) / (4.0 * math.pi)]
