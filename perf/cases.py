"""Performance cases: the work that a program using this package has it do.

Every case calls the package's public entry points (`Solver`, `BatchedSolver`,
`learned_guess.Net`) on seeded synthetic inputs that live on the GPU.  The
kinds and what they stand for:

  solve        one tensor-product solve X = (A_h + shift I)^-1 R: a
               preconditioner or a single Poisson-like solve inside a larger
               program; at 63^2 the call is a few launches of latency.
  iterate      a fixed number of quasi-Newton steps from U_0 = 0 (from a
               perturbed state with Neumann data), finite differences, 2D and
               3D, cubic / quasi-linear / 2-component problems, Dirichlet or
               Neumann data, FP64 / FP32 / split-bf16 transforms.
  sem          the same with Q^k spectral elements.
  eigen        steps of the nonlinear eigenproblem with a potential.
  grayscott    damped steps of the steady Gray-Scott system (its solves take
               thousands of steps on small grids).
  batched      many uneven 2D instances in one call (hipGraph replay).
  guess        the learned initial guess of one 2D source (two solves, the
               network in its FP16 form, the residual test).
  train        loss and gradient of one mini-batch of the guess network.

Step counts are fixed (rtol = 0), so that a pass is the same work whatever
the rounding.  Grid sides are those of the repository's own workloads (63,
127, 255, 511, 1023 interior points; 200, 400, 800, 1600 nodes) or ragged.
"""

import math

import numpy as np
import torch

import paper_2502_03611_amd as qn
from paper_2502_03611_amd import learned_guess as lg
from paper_2502_03611_amd.batched import BatchedSolver

DEV = "cuda"
BATCH_SIDES = (63, 127, 255, 511, 1023)
GS = (2.5e-4, 5e-4, 0.04, 0.065)  # D_A, D_S, rho, mu
GUESS_CHANNELS = ((2, 32), (32, 32), (32, 32), (32, 32), (32, 1))


def listed():
    return [
        # the smallest call: one solve of a 2D grid, launch latency
        {"name": "solve_63_fp64", "kind": "solve", "shape": "63x63", "ncomp": 1,
         "precision": "fp64"},
        # one 3D solve of a 2-component field on a ragged grid, FP32 transforms
        {"name": "solve_3d_ragged_sys_fp32", "kind": "solve", "shape": "150x203x176", "ncomp": 2,
         "precision": "fp32"},
        # an ordinary 2D problem solved alone: latency of many short steps
        {"name": "iterate_255_cubic_fp64", "kind": "iterate", "shape": "255x255",
         "problem": "cubic", "bc": "dirichlet", "precision": "fp64", "steps": 5},
        # the headline problem: 511^3 quasi-linear, FP64 transforms
        {"name": "iterate_511_quasilinear_fp64", "kind": "iterate", "shape": "511x511x511",
         "problem": "quasilinear", "bc": "dirichlet", "precision": "fp64", "steps": 3},
        # the same with split-bf16 transforms (the fastest time to tolerance)
        {"name": "iterate_511_quasilinear_bf16x3", "kind": "iterate", "shape": "511x511x511",
         "problem": "quasilinear", "bc": "dirichlet", "precision": "bf16x3", "steps": 3},
        # 3D Neumann problem with a potential, the tables' 200 nodes per axis
        {"name": "iterate_200_neumann_potential_fp64", "kind": "iterate", "shape": "200x200x200",
         "problem": "potential", "bc": "neumann", "precision": "fp64", "steps": 4},
        # spectral elements of order 2 (128 elements per axis)
        {"name": "sem_255_q2_fp64", "kind": "sem", "shape": "255x255x255", "order": 2,
         "bc": "dirichlet", "precision": "fp64", "steps": 3},
        # nonlinear eigenproblem, the smallest size of its table
        {"name": "eigen_200_fp64", "kind": "eigen", "shape": "200x200x200", "precision": "fp64",
         "steps": 4},
        # damped Gray-Scott steps on the smallest size of its table
        {"name": "grayscott_200_fp64", "kind": "grayscott", "side": 200, "precision": "fp64",
         "steps": 50},
        # uneven batch, half scalar and half 2-component instances
        {"name": "batched_64_fp32", "kind": "batched", "count": 64, "max_side": 1023,
         "nested": True, "precision": "fp32", "steps": 6},
        # learned initial guess of one source
        {"name": "guess_255_fp32", "kind": "guess", "side": 255, "precision": "fp32"},
        # one training mini-batch of the guess network
        {"name": "train_255_batch16", "kind": "train", "side": 255, "batch": 16},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _side(rng, lo, hi, nested):
    """A grid side in [lo, hi]: nested grids have 2^k - 1 interior points."""
    if nested:
        ks = [k for k in range(4, 12) if lo <= 2 ** k - 1 <= hi]
        return 2 ** rng.choice(ks) - 1
    return _log_int(rng, lo, hi)


def _shape(rng, dim, lo, hi, points):
    while True:
        nested = rng.random() < 0.5
        s = [_side(rng, lo, hi, nested) for _ in range(dim)]
        if math.prod(s) <= points:
            return "x".join(str(v) for v in s)


def draw(rng):
    """Half of the drawn grids have sides 2^k - 1 (nested refinements, as in the
    repository's own Dirichlet workloads), half any side of the range."""
    kind = rng.choice(["solve", "iterate", "iterate", "iterate", "sem", "eigen", "grayscott",
                       "batched", "guess", "train"])
    prec = rng.choice(["fp64", "fp64", "fp32", "bf16x3"])
    prec2 = rng.choice(["fp64", "fp64", "fp32"])
    dim = rng.choice([2, 3, 3])
    lo, hi, pts = (31, 2047, 2 ** 22) if dim == 2 else (31, 511, 400 ** 3)
    if kind == "solve":
        return {"kind": kind, "shape": _shape(rng, dim, lo, hi, pts), "ncomp": rng.choice([1, 2]),
                "precision": prec}
    if kind == "iterate":
        prob = rng.choice(["cubic", "quasilinear", "system", "potential"])
        bc = "neumann" if prob == "potential" else "dirichlet"
        return {"kind": kind, "shape": _shape(rng, dim, lo, hi, pts), "problem": prob, "bc": bc,
                "precision": prec2 if prob == "potential" else prec, "steps": rng.randint(2, 5)}
    if kind == "sem":
        order = rng.choice([2, 3, 4])
        bc = rng.choice(["dirichlet", "dirichlet", "neumann"])
        el = [_log_int(rng, 12, 255 // order) for _ in range(dim)]
        s = [e * order + (1 if bc == "neumann" else -1) for e in el]
        return {"kind": kind, "shape": "x".join(map(str, s)), "order": order, "bc": bc,
                "precision": prec2, "steps": rng.randint(2, 4)}
    if kind == "eigen":
        return {"kind": kind, "shape": _shape(rng, dim, 31, 400, 240 ** 3), "precision": prec2,
                "steps": rng.randint(2, 6)}
    if kind == "grayscott":
        return {"kind": kind, "side": _log_int(rng, 65, 800), "precision": "fp64",
                "steps": rng.randint(20, 60)}
    if kind == "batched":
        return {"kind": kind, "count": _log_int(rng, 4, 64), "max_side": _log_int(rng, 127, 1023),
                "nested": rng.random() < 0.5, "precision": rng.choice(["fp64", "fp32"]),
                "steps": rng.randint(3, 8)}
    if kind == "guess":
        return {"kind": kind, "side": _log_int(rng, 100, 400), "precision": prec2}
    return {"kind": "train", "side": _log_int(rng, 63, 255), "batch": rng.choice([4, 8, 16])}


# ---------------------------------------------------------------- inputs

def _dims(case):
    return tuple(int(v) for v in case["shape"].split("x"))


def _coords(n, a, b, closed):
    if closed:
        return a + (b - a) * torch.arange(n, dtype=torch.float64, device=DEV) / (n - 1)
    return a + (b - a) * torch.arange(1, n + 1, dtype=torch.float64, device=DEV) / (n + 1)


def _outer(factors):
    """Tensor product of per-axis vectors (array-axis order)."""
    out = factors[0]
    for f in factors[1:]:
        out = out.unsqueeze(-1) * f
    return out.contiguous()


def _outer_sum(terms):
    out = terms[0]
    for f in terms[1:]:
        out = out.unsqueeze(-1) + f
    return out.contiguous()


def _smooth(shape, rng, modes=4, closed=False):
    """A seeded smooth field: a rank-3 sum of products of short 1D series (sines
    for Dirichlet grids, cosines for closed ones), largest magnitude about 1."""
    total = None
    for _ in range(3):
        fac = []
        for n in shape:
            t = _coords(n, 0.0, 1.0, closed)
            a = rng.uniform(-1.0, 1.0, modes)
            v = torch.zeros_like(t)
            for m in range(modes):
                w = (m if closed else m + 1) * math.pi
                v = v + float(a[m]) * (torch.cos(w * t) if closed else torch.sin(w * t))
            fac.append(v)
        term = _outer(fac)
        total = term if total is None else total + term
    return total / total.abs().max()


def _quasilinear_source(shape, amp):
    """f = -div((1 + u^2) grad u) for u = amp prod sin(pi x_a)."""
    s = [torch.sin(math.pi * _coords(n, 0.0, 1.0, False)) for n in shape]
    c = [torch.cos(math.pi * _coords(n, 0.0, 1.0, False)) for n in shape]
    d = len(shape)
    u = amp * _outer(s)
    f = d * math.pi ** 2 * u * (1.0 + u * u)
    for ax in range(d):
        g = (amp * math.pi) * _outer([c[i] if i == ax else s[i] for i in range(d)])
        f -= 2.0 * u * g * g
    return f


def _grf(n, ell, rng):
    """Gaussian random field with zero boundary on the n x n grid, unit variance."""
    k = torch.arange(1, n + 1, dtype=torch.float64, device=DEV)
    w = torch.exp(-0.25 * (ell * math.pi * k) ** 2)
    m = min(n, int(8.0 / ell) + 1)  # the weights beyond underflow
    xi = torch.from_numpy(rng.standard_normal((m, m))).to(DEV)
    b = torch.sin(math.pi / (n + 1) * ((k[:, None] * k[None, :m]) % (2 * (n + 1))))
    f = b @ (w[:m, None] * xi * w[None, :m]) @ b.T
    return f / f.pow(2).mean().sqrt()


def _potential(shape, a, b, closed):
    terms = []
    for n in shape:
        x = _coords(n, a, b, closed)
        terms.append(100.0 * torch.sin(math.pi * x / 4.0) ** 2 + x * x)
    return _outer_sum(terms)


def _iterate_inputs(case, seed):
    """(U0, F, V) of an iterate or sem case, leading component axis."""
    shape = _dims(case)
    rng = np.random.default_rng(seed)
    prob = case.get("problem", "cubic")
    if prob == "quasilinear":
        f = _quasilinear_source(shape, float(rng.uniform(0.5, 2.0)))[None]
        return torch.zeros_like(f), f, None
    if prob == "potential":  # -Lap u + 10 u + 10 u^3 + V u = f on [-1, 1]^d
        c = [torch.cos(math.pi * _coords(n, -1.0, 1.0, True)) for n in shape]
        u = _outer_sum(c)
        v = _potential(shape, -1.0, 1.0, True)
        f = math.pi ** 2 * u + 10.0 * u + 10.0 * u ** 3 + v * u
        u0 = u + 0.1 * _smooth(shape, rng, closed=True)
        return u0[None].contiguous(), f[None].contiguous(), v
    closed = case["bc"] == "neumann"
    ncomp = 2 if prob == "system" else 1
    amp = float(rng.uniform(100.0, 300.0))
    f = torch.stack([amp * _smooth(shape, rng, closed=closed) for _ in range(ncomp)])
    return torch.zeros_like(f), f, None


def _sem_lin(case):
    return 1.0 if case["bc"] == "neumann" else 0.0


def _iterate_solver(case, pot):
    shape = _dims(case)
    if case["kind"] == "sem":
        return qn.Solver(shape, "cubic", beta_mode="midpoint", precision=case["precision"],
                         boundary=case["bc"], length=1.0, lin=_sem_lin(case),
                         discretization="sem", sem_order=case["order"])
    prob = case["problem"]
    if prob == "quasilinear":
        return qn.Solver(shape, "quasilinear", beta=0.0, precision=case["precision"])
    if prob == "potential":
        return qn.Solver(shape, "cubic", beta_mode="midpoint", precision=case["precision"],
                         boundary="neumann", lin=10.0, cub=10.0, potential=pot)
    return qn.Solver(shape, prob, beta_mode="midpoint", precision=case["precision"])


def _eigen_inputs(case, seed):
    shape = _dims(case)
    rng = np.random.default_rng(seed)
    v = _potential(shape, -8.0, 8.0, False)
    g = _outer([torch.exp(-0.5 * _coords(n, -8.0, 8.0, False) ** 2) for n in shape])
    u0 = g * (1.0 + 0.3 * _smooth(shape, rng))
    return u0[None].contiguous(), v


def _grayscott_inputs(case, seed):
    n = case["side"]
    rng = np.random.default_rng(seed)
    x = torch.linspace(0.0, 1.0, n, dtype=torch.float64, device=DEV)
    r = float(rng.uniform(0.18, 0.25))
    m = ((x[None, :] - 0.5) ** 2 + (x[:, None] - 0.5) ** 2 < r * r).to(torch.float64)
    u0 = torch.stack([0.25 * m, 1.0 - 0.5 * m])
    f = torch.zeros_like(u0)
    f[1] = GS[2]
    return u0, f


def _batched_sides(case):
    """Sides of the batch's instances: a property of the case, not of the seed."""
    rng = np.random.default_rng(7000 + 13 * case["count"] + case["max_side"])
    hi = case["max_side"]
    if case["nested"]:
        sides = [s for s in BATCH_SIDES if s <= hi]
        return [int(rng.choice(sides)) for _ in range(case["count"])]
    pick = [int(round(math.exp(rng.uniform(math.log(31), math.log(hi))))) for _ in range(6)]
    return [int(rng.choice(pick)) for _ in range(case["count"])]


def _batched_inputs(case, seed):
    out = []
    for i, n in enumerate(_batched_sides(case)):
        rng = np.random.default_rng([seed, i])
        out.append(torch.stack([_grf(n, 0.1, rng) for _ in range(1 + i % 2)]))
    return out


def _guess_source(n, rng):
    ell, amp = float(rng.uniform(0.05, 0.3)), float(rng.uniform(1.0, 50.0))
    return amp * _grf(n, ell, rng)


def _theta():
    return np.load(lg.WEIGHTS, allow_pickle=False)


def prepare(case, seed):
    kind = case["kind"]
    st = {"kind": kind, "case": case}
    if kind == "solve":
        shape = _dims(case)
        prob = "system" if case["ncomp"] == 2 else "cubic"
        g = torch.Generator(device=DEV).manual_seed(seed)
        st["R"] = torch.randn((case["ncomp"],) + shape, generator=g, dtype=torch.float64, device=DEV)
        st["solver"] = qn.Solver(shape, prob, beta=1.0, precision=case["precision"])
        st["X"] = torch.empty_like(st["R"])
    elif kind in ("iterate", "sem"):
        st["U0"], st["F"], st["V"] = _iterate_inputs(case, seed)
        st["solver"] = _iterate_solver(case, st["V"])
        st["U"] = torch.empty_like(st["U0"])
    elif kind == "eigen":
        st["U0"], st["V"] = _eigen_inputs(case, seed)
        st["solver"] = qn.Solver(_dims(case), "cubic", beta_mode="midpoint",
                                 precision=case["precision"], length=16.0, cub=1600.0,
                                 potential=st["V"])
        st["U"] = torch.empty_like(st["U0"])
    elif kind == "grayscott":
        st["U0"], st["F"] = _grayscott_inputs(case, seed)
        n = case["side"]
        st["solver"] = qn.Solver((n, n), "grayscott", beta_mode="midpoint", boundary="neumann",
                                 length=1.0, step=0.1, precision=case["precision"])
        st["U"] = torch.empty_like(st["U0"])
    elif kind == "batched":
        fs = _batched_inputs(case, seed)
        b = BatchedSolver([f.shape[-1] for f in fs], [f.shape[0] for f in fs],
                          precision=case["precision"], beta_mode="midpoint")
        st["solver"], st["F"], st["U"] = b, b.pool(), b.pool()
        for i, f in enumerate(fs):
            b.view(st["F"], i).copy_(f)
    elif kind == "guess":
        n = case["side"]
        st["net"] = lg.Net(n, n, max_batch=1)
        st["net"].set_params(_theta())
        st["net"].set_inference("fp16")
        st["solver"] = qn.Solver((n, n), "cubic", beta_mode="midpoint", precision=case["precision"])
        st["f"] = _guess_source(n, np.random.default_rng(seed)).contiguous().view(1, n, n)
        st["tmp"] = torch.empty_like(st["f"])
        st["red"] = torch.empty(4, dtype=torch.float64, device=DEV)
        st["used"] = torch.empty(1, dtype=torch.int32, device=DEV)
    else:
        n, bsz = case["side"], case["batch"]
        st["net"] = lg.Net(n, n, max_batch=bsz)
        st["net"].set_params(_theta())
        st["f"], st["v"], st["g"] = _train_inputs(case, seed)
    return st


def _train_inputs(case, seed):
    """Sources f, v = A_h^-1 f and the target v^3 (the nonlinear term at a
    small-amplitude solution); plain torch."""
    n = case["side"]
    rng = np.random.default_rng(seed)
    f = torch.stack([_guess_source(n, rng) for _ in range(case["batch"])])
    ax = _axis_modes(n, "dirichlet", 1.0)
    v = _solve64(f, [ax, ax], 1.0, 0.0)
    return f.contiguous(), v.contiguous(), (v ** 3).contiguous()


def run(st):
    kind, case = st["kind"], st["case"]
    if kind == "solve":
        return st["solver"].fdm_solve(st["R"], 1.0, 1.0, X=st["X"])
    if kind in ("iterate", "sem", "grayscott"):
        st["U"].copy_(st["U0"])
        r = st["solver"].iterate(st["U"], st["F"], rtol=0.0, max_iter=case["steps"])
        return {"U": st["U"], "relres": r["relres"], "iters": r["iters"]}
    if kind == "eigen":
        st["U"].copy_(st["U0"])
        r = st["solver"].eigen_iterate(st["U"], rtol=0.0, max_iter=case["steps"])
        return {"U": st["U"], "lam": r["lam"], "iters": r["iters"]}
    if kind == "batched":
        st["U"].zero_()
        _, res = st["solver"].iterate(st["U"], st["F"], rtol=0.0, max_iter=case["steps"])
        return {"U": st["U"], "iters": np.array([r["iters"] for r in res])}
    if kind == "guess":
        u0, used = lg.initial_guess_c(st["net"], st["solver"], st["f"], st["tmp"], st["red"],
                                      st["used"])
        return {"U0": u0, "used": used}
    loss = st["net"].loss_grad(st["f"], st["v"], st["g"])
    return {"loss": loss, "grad": st["net"].get_grads()}


# ---------------------------------------------------------------- least work

def _transform_flops(shape):
    """Both directions of the eigen-transforms along every axis: a fast sine or
    cosine transform of n points takes about 2.5 n log2 n operations."""
    pts = math.prod(shape)
    return 2.0 * pts * sum(2.5 * math.log2(n + 1) for n in shape)


def work(case):
    """Per step: the fields read once and written once, one transform pair and
    about ten operations per point and axis for the stencil."""
    kind = case["kind"]
    if kind == "batched":
        by = fl = 0.0
        for i, n in enumerate(_batched_sides(case)):
            c = 1 + i % 2
            by += c * n * n * 24.0
            fl += c * (_transform_flops((n, n)) + 20.0 * n * n)
        return {"bytes": by * case["steps"], "flops": fl * case["steps"]}
    if kind in ("guess", "train"):
        n = case["side"]
        px = n * n * case.get("batch", 1)
        conv = 2.0 * 9 * sum(a * b for a, b in GUESS_CHANNELS) * px
        if kind == "train":
            return {"bytes": 24.0 * px, "flops": 3.0 * conv}
        return {"bytes": 16.0 * px, "flops": conv + 2.0 * _transform_flops((n, n)) + 20.0 * px}
    shape = (case["side"],) * 2 if kind == "grayscott" else _dims(case)
    pts = math.prod(shape)
    if kind == "solve":
        c = case["ncomp"]
        return {"bytes": 16.0 * c * pts, "flops": c * _transform_flops(shape)}
    c = 2 if kind == "grayscott" or case.get("problem") == "system" else 1
    extra = 8.0 if case.get("problem") == "potential" else 0.0  # V
    per = (24.0 + extra) * c * pts
    st = 10.0 * len(shape)
    if kind == "sem":
        st = 2.0 * len(shape) * (2 * case["order"] + 1)
    return {"bytes": per * case["steps"],
            "flops": case["steps"] * c * (_transform_flops(shape) + st * pts)}


# ---------------------------------------------------------------- 64-bit values

def _axis_modes(n, bc, length):
    """(T, lam, T^-1) of the 1D finite-difference stiffness matrix."""
    j = torch.arange(n, dtype=torch.int64, device=DEV)
    if bc == "dirichlet":
        m = n + 1
        red = ((j[:, None] + 1) * (j[None, :] + 1)) % (2 * m)
        t = math.sqrt(2.0 / m) * torch.sin(math.pi / m * red.to(torch.float64))
        lam = 4.0 * (m / length) ** 2 * torch.sin(math.pi / (2 * m) * (j + 1).to(torch.float64)) ** 2
        return t, lam, t
    m = n - 1
    red = (j[:, None] * j[None, :]) % (2 * m)
    t = torch.cos(math.pi / m * red.to(torch.float64))
    lam = 4.0 * (m / length) ** 2 * torch.sin(math.pi / (2 * m) * j.to(torch.float64)) ** 2
    w = torch.ones(n, dtype=torch.float64, device=DEV)
    w[0] = w[-1] = 0.5
    return t, lam, (2.0 / m) * w[:, None] * t.T * w[None, :]


def _sem_modes(n, order, bc, length):
    """(T, lam, T^-1, H) of Gauss-Lobatto elements with the lumped mass."""
    leg = np.polynomial.legendre
    c = np.zeros(order + 1)
    c[order] = 1.0
    inner = np.sort(leg.legroots(leg.legder(c))) if order > 1 else np.array([])
    for _ in range(3):  # polish the roots of P_k'
        if inner.size:
            inner = inner - leg.legval(inner, leg.legder(c)) / leg.legval(inner, leg.legder(c, 2))
    x = np.concatenate([[-1.0], inner, [1.0]])
    w = 2.0 / (order * (order + 1) * leg.legval(x, c) ** 2)
    d = np.zeros((order + 1, order + 1))
    for p in range(order + 1):
        for q in range(order + 1):
            if p != q:
                num = np.prod([x[q] - x[m] for m in range(order + 1) if m not in (p, q)])
                d[q, p] = num / np.prod([x[p] - x[m] for m in range(order + 1) if m != p])
    d[np.arange(order + 1), np.arange(order + 1)] = -d.sum(axis=1)
    el = (n + 1) // order if bc == "dirichlet" else (n - 1) // order
    jac = 0.5 * length / el
    ke = (d.T * w) @ d / jac
    tot = el * order + 1
    m, s = np.zeros(tot), np.zeros((tot, tot))
    for e in range(el):
        i = e * order + np.arange(order + 1)
        m[i] += w * jac
        s[np.ix_(i, i)] += ke
    if bc == "dirichlet":
        m, s = m[1:-1], s[1:-1, 1:-1]
    r = 1.0 / np.sqrt(m)
    lam, q = np.linalg.eigh(r[:, None] * s * r[None, :])
    conv = [r[:, None] * q, lam, q.T / r[None, :], s / m[:, None]]
    return tuple(torch.from_numpy(np.ascontiguousarray(v)).to(DEV) for v in conv)


def _apply(mat, x, axis):
    """Mode product: mat along one axis of x."""
    y = x.movedim(axis, -1)
    return (y.reshape(-1, y.shape[-1]) @ mat.T).reshape(y.shape).movedim(-1, axis)


def _solve64(r, axes, scale, shift):
    """(scale A + shift I)^-1 r over the last len(axes) axes (array-axis order)."""
    d = len(axes)
    y = r
    for a in range(d):
        y = _apply(axes[a][2], y, a - d)
    y = y / (scale * _outer_sum([ax[1] for ax in axes]) + shift)
    for a in range(d):
        y = _apply(axes[a][0], y, a - d)
    return y.contiguous()


def _shift(u, axis, step, bc):
    """u at the neighbouring node along one axis (zero or mirrored beyond the ends)."""
    n = u.shape[axis]
    idx = torch.arange(n, device=u.device) + step
    if bc == "neumann":
        idx = torch.where(idx < 0, -idx, idx)
        idx = torch.where(idx > n - 1, 2 * (n - 1) - idx, idx)
        return u.index_select(axis, idx)
    out = torch.zeros_like(u)
    if n > 1:
        src, dst = (slice(1, n), slice(0, n - 1)) if step > 0 else (slice(0, n - 1), slice(1, n))
        out.movedim(axis, 0)[dst] = u.movedim(axis, 0)[src]
    return out


def _lap(u, dim, bc, length):
    """A_h u over the last `dim` axes."""
    out = torch.zeros_like(u)
    for a in range(-dim, 0):
        n = u.shape[a]
        ih2 = ((n + 1 if bc == "dirichlet" else n - 1) / length) ** 2
        out += ih2 * (2.0 * u - _shift(u, a, 1, bc) - _shift(u, a, -1, bc))
    return out


def _quasilinear(u, dim):
    a = 1.0 + u * u
    out = torch.zeros_like(u)
    for ax in range(-dim, 0):
        ih2 = float(u.shape[ax] + 1) ** 2
        for s in (1, -1):
            un = _shift(u, ax, s, "dirichlet")
            out += (0.5 * ih2) * (a + 1.0 + un * un) * (u - un)
    return out


def _mid(lo, hi):
    return 0.5 * (float(lo.min()) + float(hi.max()))


def _residual64(prob, u, f, v, dim, sem, bc, length, lin, cub):
    """(R, scale, shift) at u."""
    if prob == "quasilinear":
        a = 1.0 + u * u
        return _quasilinear(u, dim) - f, _mid(a, a), 0.0
    if prob == "grayscott":
        da, ds, rho, mu = GS
        a, s = u[0], u[1]
        lap = _lap(u, 2, "neumann", 1.0)
        r = torch.stack([da * lap[0] - s * a * a + (mu + rho) * a - f[0],
                         ds * lap[1] + s * a * a + rho * s - f[1]])
        p, q = -2.0 * s * a + mu + rho, a * a + rho
        disc = torch.sqrt(torch.clamp((p - q) ** 2 - 8.0 * s * a ** 3, min=0.0))
        return r, 1.0, _mid(0.5 * (p + q - disc), 0.5 * (p + q + disc))
    if sem is not None:
        lap = sum(_apply(sem[ax][3], u, ax - dim) for ax in range(dim))
    else:
        lap = _lap(u, dim, bc, length)
    if prob == "system":
        r = lap + u ** 3 - u.flip(0) - f
        p, q = 3.0 * u[0] ** 2, 3.0 * u[1] ** 2
        disc = torch.sqrt((p - q) ** 2 + 4.0)
        return r, 1.0, _mid(0.5 * (p + q - disc), 0.5 * (p + q + disc))
    r = lap + lin * u + cub * u ** 3 - f
    d = 3.0 * cub * u * u + lin
    if v is not None:
        r, d = r + v * u, d + v
    return r, 1.0, _mid(d, d)


def _iterate64(prob, u, f, v, axes, steps, bc, length=1.0, lin=0.0, cub=1.0, sem=False, tau=1.0):
    dim = len(axes)
    args = (f, v, dim, axes if sem else None, bc, length, lin, cub)
    for _ in range(steps):
        r, c, b = _residual64(prob, u, *args)
        if prob == "grayscott":
            du = torch.stack([_solve64(r[k], axes, GS[k], b) for k in range(2)])
        else:
            du = _solve64(r, axes, c, b)
        u = u - tau * du
    r = _residual64(prob, u, *args)[0]
    return u, float(r.pow(2).sum().sqrt() / f.pow(2).sum().sqrt())


def _eigen64(u, v, axes, steps):
    dim = len(axes)
    hd = math.prod(16.0 / (n + 1) for n in u.shape[-dim:])

    def state(w):
        w = w / (hd * w.pow(2).sum()).sqrt()
        g = _lap(w, dim, "dirichlet", 16.0) + 1600.0 * w ** 3 + v * w
        return w, g, float(hd * (g * w).sum())

    w, g, lam = state(u)
    for _ in range(steps):
        d = 4800.0 * w * w + v
        w, g, lam = state(w - _solve64(g - lam * w, axes, 1.0, _mid(d, d) - lam))
    return w, lam


def _net64(theta, f, v):
    """g = net(f / 50, v): 3x3 'same' cross-correlations as nine shifted products."""
    bsz, h, w = f.shape
    x = torch.stack([f / 50.0, v]).reshape(2, -1)
    p = 0
    for li, (ci, co) in enumerate(GUESS_CHANNELS):
        wt = theta[p:p + co * ci * 9].reshape(co, ci, 3, 3)
        bias = theta[p + co * ci * 9:p + co * ci * 9 + co]
        p += co * ci * 9 + co
        pad = torch.nn.functional.pad(x.reshape(ci, bsz, h, w), (1, 1, 1, 1))
        y = bias[:, None].expand(co, bsz * h * w)
        for dy in range(3):
            for dx in range(3):
                y = y + wt[:, :, dy, dx] @ pad[:, :, dy:dy + h, dx:dx + w].reshape(ci, -1)
        x = y if li == 4 else 0.5 * y * (1.0 + torch.erf(y * math.sqrt(0.5)))
    return x.reshape(bsz, h, w)


def exact(case, seed):
    kind = case["kind"]
    if kind == "solve":
        shape = _dims(case)
        g = torch.Generator(device=DEV).manual_seed(seed)
        r = torch.randn((case["ncomp"],) + shape, generator=g, dtype=torch.float64, device=DEV)
        return _solve64(r, [_axis_modes(n, "dirichlet", 1.0) for n in shape], 1.0, 1.0)
    if kind in ("iterate", "sem"):
        shape = _dims(case)
        u0, f, v = _iterate_inputs(case, seed)
        prob, k = case.get("problem", "cubic"), case["steps"]
        if kind == "sem":
            axes = [_sem_modes(n, case["order"], case["bc"], 1.0) for n in shape]
            u, rel = _iterate64("cubic", u0, f, None, axes, k, case["bc"], lin=_sem_lin(case),
                                sem=True)
        elif prob == "potential":
            axes = [_axis_modes(n, "neumann", 2.0) for n in shape]
            u, rel = _iterate64("cubic", u0, f, v, axes, k, "neumann", 2.0, 10.0, 10.0)
        else:
            axes = [_axis_modes(n, "dirichlet", 1.0) for n in shape]
            u, rel = _iterate64(prob, u0, f, None, axes, k, "dirichlet")
        return {"U": u, "relres": rel, "iters": k}
    if kind == "grayscott":
        u0, f = _grayscott_inputs(case, seed)
        ax = _axis_modes(case["side"], "neumann", 1.0)
        u, rel = _iterate64("grayscott", u0, f, None, [ax, ax], case["steps"], "neumann", tau=0.1)
        return {"U": u, "relres": rel, "iters": case["steps"]}
    if kind == "eigen":
        u0, v = _eigen_inputs(case, seed)
        axes = [_axis_modes(n, "dirichlet", 16.0) for n in _dims(case)]
        u, lam = _eigen64(u0, v, axes, case["steps"])
        return {"U": u, "lam": lam, "iters": case["steps"]}
    if kind == "batched":
        fs = _batched_inputs(case, seed)
        b = BatchedLayout([f.shape[-1] for f in fs], [f.shape[0] for f in fs])
        pool = torch.zeros(b.elems, dtype=torch.float64, device=DEV)
        modes = {}
        for i, f in enumerate(fs):
            n = f.shape[-1]
            if n not in modes:
                modes[n] = _axis_modes(n, "dirichlet", 1.0)
            prob = "system" if f.shape[0] == 2 else "cubic"
            u, _ = _iterate64(prob, torch.zeros_like(f), f, None, [modes[n]] * 2, case["steps"],
                              "dirichlet")
            b.view(pool, i).copy_(u)
        return {"U": pool, "iters": np.full(len(fs), case["steps"])}
    theta = torch.from_numpy(_theta()).to(DEV, torch.float64)
    if kind == "guess":
        n = case["side"]
        f = _guess_source(n, np.random.default_rng(seed)).view(1, n, n)
        ax = _axis_modes(n, "dirichlet", 1.0)
        g = _net64(theta, f, _solve64(f, [ax, ax], 1.0, 0.0))
        u0 = _solve64(f - g, [ax, ax], 1.0, 0.0)
        r = _lap(u0, 2, "dirichlet", 1.0) + u0 ** 3 - f
        keep = bool(r.pow(2).sum() < f.pow(2).sum())
        return {"U0": u0 if keep else torch.zeros_like(u0),
                "used": torch.tensor([int(keep)], dtype=torch.int32, device=DEV)}
    f, v, tgt = _train_inputs(case, seed)
    theta.requires_grad_(True)
    loss = (_net64(theta, f, v) - tgt).pow(2).mean()
    loss.backward()
    return {"loss": float(loss.detach()), "grad": theta.grad.cpu().numpy()}


class BatchedLayout:
    """The documented pool layout of a batch: instances of equal (side, ncomp)
    form a class stored as one (ncomp, count, n, n) block, classes and members
    in the order of their first appearance."""

    def __init__(self, sides, ncomp):
        keys = list(dict.fromkeys(zip(sides, ncomp)))
        self.where = {}
        off = 0
        for n, c in keys:
            mem = [i for i, k in enumerate(zip(sides, ncomp)) if k == (n, c)]
            for s, i in enumerate(mem):
                self.where[i] = (off + s * n * n, len(mem) * n * n, n, c)
            off += c * len(mem) * n * n
        self.elems = off

    def view(self, pool, i):
        off, cs, n, c = self.where[i]
        return torch.as_strided(pool, (c, n, n), (cs, n, 1), off)


__all__ = ["listed", "draw", "prepare", "run", "work", "exact"]
