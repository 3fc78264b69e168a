"""Performance cases of the block ILU(k) framework.

The work that a reservoir or Poisson code has this framework do, through
``BlockILU``, ``BlockILUBatch``, ``autograd.solve`` and the device symbolic
phase: single applications and products (the body of a user's own Krylov
loop), refactorisation after new values, whole time steps (factorisation +
solve), several right-hand sides, the differentiable solve with its backward
pass, batches of small systems and the symbolic phase.  Grids, block sizes
and distributions are those of ``bench.py`` and ``synth.py``, the drawn ones
spread around them.

``listed()`` / ``draw(rng)`` give cases, ``prepare`` the handle and inputs of
one, ``run`` one pass, ``work`` the bytes and operations a pass cannot do
without and ``exact`` its outputs in plain 64-bit torch.
"""
from __future__ import annotations

import numpy as np
import torch

from paper_1703_01325_amd import api, autograd, synth

# Block stencil in ascending column order: (dx, dy, dz) of the 7-point grid.
STENCIL = ((0, 0, -1), (0, -1, 0), (-1, 0, 0), (0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1))
# Lower neighbours of ILU(0) and ILU(1) on it, ascending; the upper ones mirror them.
LOWER = {0: ((0, 0, -1), (0, -1, 0), (-1, 0, 0)),
         1: ((0, 0, -1), (1, 0, -1), (0, 1, -1), (0, -1, 0), (1, -1, 0), (-1, 0, 0))}


def _case(name, kind, grid, b, k, **options):
    nx, ny, nz = grid
    case = {"name": name, "kind": kind, "nx": nx, "ny": ny, "nz": nz, "b": b, "k": k}
    case.update(options)
    return case


def listed():
    layered = (60, 220, 85)
    return [
        # one application on a small model: launches and latency
        _case("apply_10cube_ilu1", "apply", (10, 10, 10), 3, 1, precision="fp64"),
        # the preconditioner inside a user's own iteration, full-size model
        _case("apply_layered_ilu0", "apply", layered, 3, 0, precision="fp64"),
        # the same with the stronger factorisation, stored in FP32
        _case("apply_layered_ilu1_fp32", "apply", layered, 3, 1, precision="fp32"),
        # the product beside it
        _case("spmv_layered", "spmv", layered, 3, 0),
        # new values in a kept structure: refactor and hand the factors to the caller
        _case("factor_64cube_ilu1", "factor", (64, 64, 64), 3, 1, precision="fp64"),
        # a whole time step of the full-size model: factorisation and BiCGSTAB to 1e-8
        _case("step_layered_ilu0", "step", layered, 3, 0, precision="fp64", method="bicgstab", rhs=1),
        # many right-hand sides of one factored model
        _case("solve_64cube_ilu1_rhs32", "solve", (64, 64, 64), 3, 1, precision="fp64", method="bicgstab", rhs=32),
        # the 120^3 Poisson matrix in blocks of 2, GMRES(20) to 1e-6
        _case("gmres_poisson120_b2_ilu1", "poisson", (60, 120, 120), 2, 1, precision="fp64"),
        # differentiable solve of a four-unknown model: forward and backward pass
        _case("adjoint_64cube_b4_ilu0", "adjoint", (64, 64, 64), 4, 0),
        # independent small systems of mixed sizes and block sizes, solved together
        _case("batch_solve_64", "batch", (0, 0, 0), 0, 0, systems=64, side_lo=8, side_hi=40),
        # a new structure: symbolic phase and level sets of both sweeps
        _case("symbolic_layered_ilu1", "symbolic", layered, 1, 1),
        # large blocks: factorisation and solve of a small grid of 25 unknowns a cell
        _case("step_12cube_b25_ilu0", "step", (12, 12, 12), 25, 0, precision="fp64", method="bicgstab", rhs=1),
    ]


def _drawn_grid(rng, lo, hi):
    """Three sides whose product lies in about [lo, hi], uniform in its
    logarithm, the sides up to a factor of about two apart."""
    cells = lo * (hi / lo) ** rng.random()
    skew = [2.0 ** rng.uniform(-0.6, 0.6) for _ in range(3)]
    scale = (cells / (skew[0] * skew[1] * skew[2])) ** (1.0 / 3.0)
    return tuple(max(3, int(round(scale * s))) for s in skew)


def draw(rng):
    kind = rng.choice(["apply", "apply", "spmv", "factor", "step", "solve", "poisson", "adjoint", "batch",
                       "symbolic", "large"])
    b = rng.choice([1, 2, 3, 3, 4, 5, 6, 8])
    k = rng.choice([0, 1])
    precision = rng.choice(["fp64", "fp64", "fp32"])
    big = 1_100_000 * 9 // max(9, b * b)
    if kind in ("apply", "factor"):
        case = _case("", kind, _drawn_grid(rng, 900, big), b, k, precision=precision)
    elif kind == "spmv":
        case = _case("", kind, _drawn_grid(rng, 900, big), b, 0)
    elif kind == "step":
        case = _case("", kind, _drawn_grid(rng, 900, big), b, k, precision=precision,
                     method=rng.choice(["bicgstab", "bicgstab", "orthomin"]), rhs=1)
    elif kind == "solve":
        case = _case("", kind, _drawn_grid(rng, 900, 250_000 * 9 // max(9, b * b)), b, k, precision=precision,
                     method="bicgstab", rhs=rng.choice([2, 3, 5, 8, 8, 16, 24, 32]))
    elif kind == "poisson":
        k = rng.choice([0, 1, 2, 3])
        b = rng.choice([1, 2, 4, 8])
        gx, gy, gz = _drawn_grid(rng, 8000, 1_700_000 if k < 2 else 300_000)
        case = _case("", kind, (max(4, (gx + b - 1) // b), gy, gz), b, k, precision="fp64")
    elif kind == "adjoint":
        case = _case("", kind, _drawn_grid(rng, 900, 262_144 * 16 // max(16, b * b)), b, k)
    elif kind == "batch":
        case = _case("", kind, (0, 0, 0), 0, 0, systems=rng.randint(5, 64), side_lo=rng.choice([5, 8, 11]),
                     side_hi=rng.choice([16, 25, 40]))
    elif kind == "symbolic":
        case = _case("", kind, _drawn_grid(rng, 20_000, 1_100_000), 1, rng.choice([0, 1, 1, 2]))
    else:
        case = _case("", "step", _drawn_grid(rng, 200, 1700), rng.choice([9, 12, 16, 21, 25]), 0, precision="fp64",
                     method="bicgstab", rhs=1)
    del case["name"]
    return case


# ---------------------------------------------------------------------------
# Inputs, as dense stencils: A[cell, slot, r, c], slots in STENCIL order
# ---------------------------------------------------------------------------
def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _uniform(gen, *shape, lo=-1.0, hi=1.0):
    return torch.rand(*shape, generator=gen, device="cuda", dtype=torch.float64) * (hi - lo) + lo


class _Grid:
    """Cells in natural order (x fastest) and their stencil neighbours."""

    def __init__(self, nx, ny, nz):
        self.shape = (nx, ny, nz)
        self.nb = nx * ny * nz
        cell = torch.arange(self.nb, device="cuda")
        self.x = cell % nx
        self.y = torch.div(cell, nx, rounding_mode="floor") % ny
        self.z = torch.div(cell, nx * ny, rounding_mode="floor")
        self.valid = torch.stack([self.inside(o) for o in STENCIL], 1)
        self.cols = torch.stack([cell + self.linear(o) for o in STENCIL], 1).clamp_(0, self.nb - 1)

    def linear(self, o):
        return o[0] + self.shape[0] * (o[1] + self.shape[1] * o[2])

    def inside(self, o):
        m = torch.ones(self.nb, dtype=torch.bool, device="cuda")
        for c, d, n in zip((self.x, self.y, self.z), o, self.shape):
            if d:
                m &= (c + d >= 0) & (c + d < n)
        return m


def _reservoir(g, b, gen, layered, sigma):
    """Lognormal permeability (a mean per layer if `layered`), two-point
    transmissibilities, full blocks, row-diagonally dominant."""
    nz = g.shape[2]
    mu = _uniform(gen, nz, lo=-2.0, hi=3.0)[g.z] if layered else 0.0
    K = torch.exp(mu + sigma * torch.randn(g.nb, generator=gen, device="cuda", dtype=torch.float64))
    A = 0.1 * torch.randn(g.nb, 7, b, b, generator=gen, device="cuda", dtype=torch.float64)
    Kn = K[g.cols]
    T = 2.0 * K[:, None] * Kn / (K[:, None] + Kn)
    d = torch.arange(b, device="cuda")
    A[:, :, d, d] -= T[:, :, None]
    A *= g.valid[:, :, None, None]
    A[:, 3] = 0.0
    total = A.abs().sum(dim=(1, 3))
    A[:, 3] = _uniform(gen, g.nb, b, b, lo=-0.2, hi=0.2)
    A[:, 3, d, d] += total + 1.0
    return A


def _poisson(g, b):
    """The 7-point Laplacian, b consecutive unknowns of a grid line a block."""
    A = torch.zeros(g.nb, 7, b, b, device="cuda", dtype=torch.float64)
    d = torch.arange(b, device="cuda")
    A[:, 3, d, d] = 6.0
    A[:, 3, d[1:], d[:-1]] = -1.0
    A[:, 3, d[:-1], d[1:]] = -1.0
    A[:, 2, 0, b - 1] = -1.0
    A[:, 4, b - 1, 0] = -1.0
    for s in (0, 1, 5, 6):
        A[:, s, d, d] = -1.0
    return A * g.valid[:, :, None, None]


def _values(g, A):
    """The stored blocks, each column by column."""
    return A.transpose(2, 3)[g.valid].reshape(-1).contiguous()


def _product(g, A, x):
    """A x, x of shape (n,) or (n, R)."""
    b = A.shape[2]
    xb = x.reshape(g.nb, b, -1)
    y = torch.zeros_like(xb)
    for s in range(7):
        xs = xb[g.cols[:, s]]
        for c in range(b):
            y += A[:, s, :, c, None] * xs[:, c, None, :]
    return y.reshape(x.shape)


def _product_t(g, A, x):
    """A^T x, x of shape (n,)."""
    b = A.shape[2]
    xb = x.reshape(g.nb, b)
    y = torch.zeros_like(xb)
    for s in range(7):
        m = g.valid[:, 6 - s]                        # row j - offset holds slot s for column j
        i = g.cols[:, 6 - s]
        for r in range(b):
            y += torch.where(m[:, None], A[i, s, r, :], 0.0) * xb[i][:, r, None]
    return y.reshape(-1)


def _system(case, seed):
    """(grid, dense A, generator) of one system."""
    g = _Grid(case["nx"], case["ny"], case["nz"])
    gen = _generator(seed)
    if case["kind"] == "poisson":
        return g, _poisson(g, case["b"]), gen
    layered = g.nb > 300_000
    return g, _reservoir(g, case["b"], gen, layered, 1.5 if layered else 1.0 if g.nb < 50_000 else 2.0), gen


def _members(case):
    """Grids and block sizes of a batch."""
    rng = np.random.Generator(np.random.PCG64([case["systems"], case["side_lo"], case["side_hi"]]))
    out = []
    for _ in range(case["systems"]):
        sides = tuple(int(v) for v in rng.integers(case["side_lo"], case["side_hi"] + 1, size=3))
        out.append((sides, int(rng.choice(np.array(synth.BATCH_BLOCK_SIZES)))))
    return out


def _vector(case, g, gen):
    n = g.nb * case["b"]
    R = case.get("rhs", 1)
    return _uniform(gen, n) if R == 1 else _uniform(gen, n, R)


def _source(case, g, gen):
    """Right-hand side of the Poisson systems: a source of about 1 everywhere."""
    return 1.0 + 0.2 * _uniform(gen, g.nb * case["b"])


def _batch_inputs(case, seed):
    gen = _generator(seed)
    for (sides, b) in _members(case):
        g = _Grid(*sides)
        yield sides, b, g, _reservoir(g, b, gen, False, 1.0), _uniform(gen, g.nb * b)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        systems, values, rhs = [], [], []
        for sides, b, g, A, x in _batch_inputs(case, seed):
            Ap, Aj = synth.stencil7_pattern(*sides)
            systems.append((g.nb, b, Ap, Aj))
            values.append(_values(g, A))
            rhs.append(_product(g, A, x))
        M = api.BlockILUBatch(systems, case["k"])
        if M.factor(values) is not None:
            raise RuntimeError("singular pivot block")
        return {"kind": kind, "M": M, "values": values, "b": torch.cat(rhs)}
    Ap, Aj = synth.stencil7_pattern(case["nx"], case["ny"], case["nz"])
    if kind == "symbolic":
        # inactive couplings: the seed picks the lines of cells without x
        # couplings, inside the grid and four cells apart, so that as many
        # entries and levels remain whichever they are
        rng = np.random.Generator(np.random.PCG64(int(seed)))
        ys, zs = np.arange(2, case["ny"] - 2, 4), np.arange(2, case["nz"] - 2, 4)
        lines = (ys[None, :] + case["ny"] * zs[:, None]).ravel()
        cut = np.zeros(case["ny"] * case["nz"], dtype=bool)
        cut[rng.choice(lines, size=(lines.size + 1) // 3, replace=False)] = True
        rows = np.repeat(np.arange(Ap.size - 1), np.diff(Ap))
        keep = ~(cut[rows // case["nx"]] & (np.abs(Aj - rows) == 1))
        Aj = Aj[keep]
        Ap = np.concatenate([[0], np.cumsum(np.bincount(rows[keep], minlength=Ap.size - 1))]).astype(np.int32)
        return {"kind": kind, "k": case["k"], "Ap": torch.from_numpy(Ap).cuda(), "Aj": torch.from_numpy(Aj).cuda()}
    g, A, gen = _system(case, seed)
    values = _values(g, A)
    M = api.BlockILU(g.nb, case["b"], Ap, Aj, case["k"], transpose=kind == "adjoint")
    state = {"kind": kind, "M": M, "values": values, "precision": case.get("precision", "fp64"),
             "method": case.get("method", "bicgstab")}
    if kind == "spmv":
        state["x"] = _vector(case, g, gen)
        return state
    if M.factor(values, precision=state["precision"]) >= 0:
        raise RuntimeError("singular pivot block")
    if kind == "factor":
        return state
    if kind == "apply":
        state["r"] = _vector(case, g, gen)
        return state
    if kind == "poisson":
        state["b"] = _source(case, g, gen)
    else:
        state["b"] = _product(g, A, _vector(case, g, gen))
    if kind == "adjoint":
        state["values"].requires_grad_(True)
        state["b"].requires_grad_(True)
        state["grad"] = _product_t(g, A, _vector(case, g, gen))
    return state


def _solved(result):
    x, status, info = result
    return {"x": x, "status": status, "iterations": np.array([i[1] for i in info]),
            "relres": np.array([i[2] for i in info])}


def run(state):
    kind = state["kind"]
    if kind == "symbolic":
        Pp, Pj, lev = api.symbolic_device(state["Ap"], state["Aj"], state["k"])
        return [Pp, Pj, lev, *api.levels_device(Pp, Pj, 0), *api.levels_device(Pp, Pj, 1)]
    M = state["M"]
    if kind == "apply":
        return M.apply(state["r"])
    if kind == "spmv":
        return M.spmv(state["values"], state["x"])
    if kind == "factor":
        bad = M.factor(state["values"], precision=state["precision"])
        F, D = M.factors() if state["precision"] == "fp64" else M.factors_f32()
        return [F, D, bad]
    if kind == "batch":
        return _solved(M.solve(state["b"], rtol=1e-8))
    if kind == "poisson":
        return _solved(M.solve(state["values"], state["b"], method="gmres", restart=20, rtol=1e-6, maxit=4000))
    if kind == "adjoint":
        x = autograd.solve(state["values"], state["b"], M)
        dA, db = torch.autograd.grad(x, (state["values"], state["b"]), state["grad"])
        return [x.detach(), dA, db]
    if kind == "step":
        M.factor(state["values"], precision=state["precision"])
    return _solved(M.solve(state["values"], state["b"], method=state["method"], restart=10, rtol=1e-8))


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
def _blocks(case, offsets):
    n = 0
    for (dx, dy, dz) in offsets:
        n += max(0, case["nx"] - abs(dx)) * max(0, case["ny"] - abs(dy)) * max(0, case["nz"] - abs(dz))
    return n


def work(case):
    kind = case["kind"]
    if kind == "batch":
        # the members are factored already: one application and one product of each
        parts = [work({"kind": "solve", "nx": s[0], "ny": s[1], "nz": s[2], "b": b, "k": case["k"]})
                 for s, b in _members(case)]
        return {key: sum(part[key] for part in parts) for key in ("bytes", "flops")}
    b, k, R = case["b"], case["k"], case.get("rhs", 1)
    nb = case["nx"] * case["ny"] * case["nz"]
    n, bb = nb * b, b * b
    s = 4 if case.get("precision") == "fp32" else 8
    stored = _blocks(case, STENCIL)
    low = _blocks(case, LOWER[min(k, 1)])
    a_bytes = stored * (8 * bb + 4) + 4 * nb
    f_bytes = (2 * low + nb) * (s * bb + 4) + 8 * nb
    product, application = 2 * bb * stored * R, 2 * bb * (2 * low + nb) * R
    factor = 2 * b * bb * (low + nb) + 2 * b * bb * low * len(LOWER[min(k, 1)]) // 2
    if kind == "symbolic":
        # the pattern in; pattern, levels of fill and two level sets out
        return {"bytes": 4 * stored + 4 * nb + 8 * (2 * low + nb) + 20 * nb, "flops": 0}
    if kind == "spmv":
        return {"bytes": a_bytes + 16 * n, "flops": product}
    if kind == "apply":
        return {"bytes": f_bytes + 16 * n, "flops": application}
    if kind == "factor":
        return {"bytes": a_bytes + (2 * low + 2 * nb) * s * bb, "flops": factor}
    if kind == "adjoint":
        # A and the gradient of it, right-hand side, upstream gradient and three vectors out
        return {"bytes": a_bytes + f_bytes + 8 * bb * stored + 40 * n,
                "flops": 2 * (product + application) + bb * stored}
    # one application and one product at the least, of A and its factors
    return {"bytes": a_bytes + f_bytes + 16 * n * R,
            "flops": (factor if kind == "step" else 0) + product + application}


# ---------------------------------------------------------------------------
# The outputs in plain 64-bit torch
# ---------------------------------------------------------------------------
def _mul(a, b):
    return (a[:, :, :, None] * b[:, None, :, :]).sum(2)


def _inverse(a):
    """Gauss-Jordan of diagonally dominant blocks."""
    b = a.shape[1]
    w = torch.cat([a, torch.eye(b, device=a.device, dtype=a.dtype).expand_as(a)], 2)
    for p in range(b):
        row = w[:, p] / w[:, p, p, None]
        w = w - w[:, :, p, None] * row[:, None, :]
        w[:, p] = row
    return w[:, :, b:]


def _factor_exact(g, A, k):
    """Block ILU(k) factors (k = 0, 1) of the stencil matrix, level by level:
    (blocks by offset -- L below, U above --, D^{-1}, rows of each level)."""
    b = A.shape[2]
    lower = LOWER[k]
    upper = tuple(tuple(-d for d in o) for o in reversed(lower))
    kept = lower + ((0, 0, 0),) + upper
    F = {o: torch.zeros(g.nb, b, b, device="cuda", dtype=torch.float64) for o in kept}
    for s, o in enumerate(STENCIL):
        F[o] = A[:, s].clone()
    level = g.x + g.y + g.z if k == 0 else g.x + 2 * g.y + 3 * g.z
    order = torch.argsort(level, stable=True)
    sets = torch.split(order, [c for c in torch.bincount(level).tolist()])
    sets = [s for s in sets if s.numel()]
    inside = {o: g.inside(o) for o in lower}
    D = torch.zeros(g.nb, b, b, device="cuda", dtype=torch.float64)
    for rows in sets:
        for o in lower:
            i = rows[inside[o][rows]]
            if not i.numel():
                continue
            p = i + g.linear(o)
            f = _mul(F[o][i], D[p])
            F[o][i] = f
            for u in upper:
                t = tuple(c + d for c, d in zip(o, u))
                if t in F:
                    F[t][i] -= _mul(f, F[u][p])
        D[rows] = _inverse(F[(0, 0, 0)][rows])
    return F, D, sets


def _factors_exact(g, A, k):
    """The factors in pattern order, blocks column by column: L below, U' =
    D^{-1} U above, the identity on the diagonal; and D^{-1}."""
    F, D, _ = _factor_exact(g, A, k)
    b = A.shape[2]
    blocks, mask = [], []
    for o in F:
        if o == (0, 0, 0):
            blocks.append(torch.eye(b, device="cuda", dtype=torch.float64).expand(g.nb, b, b))
        else:
            blocks.append(F[o] if o in LOWER[k] else _mul(D, F[o]))
        mask.append(g.inside(o))
    P = torch.stack(blocks, 1)[torch.stack(mask, 1)]
    return [P.transpose(1, 2).reshape(-1), D.transpose(1, 2).reshape(-1)]


def _apply_exact(g, A, k, r):
    """(L D U')^{-1} r of those factors."""
    F, D, sets = _factor_exact(g, A, k)
    lower = LOWER[k]
    upper = [o for o in F if o not in lower and o != (0, 0, 0)]
    inside = {o: g.inside(o) for o in F}
    y = r.reshape(g.nb, -1).clone()
    for rows in sets:
        for o in lower:
            i = rows[inside[o][rows]]
            y[i] -= (F[o][i] * y[i + g.linear(o)][:, None, :]).sum(2)
    z = torch.zeros_like(y)
    for rows in reversed(sets):
        acc = y[rows].clone()
        for u in upper:
            m = inside[u][rows]
            i = rows[m]
            acc[m] -= (F[u][i] * z[i + g.linear(u)][:, None, :]).sum(2)
        z[rows] = (D[rows] * acc[:, None, :]).sum(2)
    return z.reshape(-1)


def _poisson_solution(case, f):
    """The Laplacian solved in its sine eigenbasis."""
    v = f.reshape(case["nz"], case["ny"], case["nx"] * case["b"])
    basis, eig = [], []
    for n in v.shape:
        i = torch.arange(1, n + 1, device="cuda", dtype=torch.float64)
        angle = i * (np.pi / (n + 1))
        basis.append(torch.sin(i[:, None] * angle[None, :]) * (2.0 / (n + 1)) ** 0.5)
        eig.append(2.0 - 2.0 * torch.cos(angle))

    def turn(w):
        for axis in range(3):
            w = torch.tensordot(basis[axis], w.movedim(axis, 0).contiguous(), dims=1).movedim(0, axis)
        return w.contiguous()

    total = eig[0][:, None, None] + eig[1][None, :, None] + eig[2][None, None, :]
    return turn(turn(v) / total).reshape(-1)


def _exact_solution(x):
    return {"x": x, "status": None, "iterations": None, "relres": None}


def exact(case, seed):
    kind = case["kind"]
    if kind == "symbolic":
        return None
    if kind == "batch":
        return _exact_solution(torch.cat([x for _, _, _, _, x in _batch_inputs(case, seed)]))
    g, A, gen = _system(case, seed)
    if kind == "factor":
        return [*_factors_exact(g, A, case["k"]), None]
    if kind == "poisson":
        return _exact_solution(_poisson_solution(case, _source(case, g, gen)))
    x = _vector(case, g, gen)
    if kind == "spmv":
        return _product(g, A, x)
    if kind == "apply":
        return _apply_exact(g, A, case["k"], x)
    if kind == "adjoint":
        lam = _vector(case, g, gen)
        b = case["b"]
        dA = -lam.reshape(g.nb, 1, 1, b) * x.reshape(g.nb, b)[g.cols][:, :, :, None]
        return [x, dA[g.valid].reshape(-1), lam]
    return _exact_solution(x)
