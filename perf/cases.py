"""The work that programs ask of this solver, as cases that can be timed.

Every case is a linear system of the implicit DG discretisation of the 2D
Euler equations (or a batch of them): the Jacobian about a smooth base state,
periodic or far-field in each direction, 4 (p+1)^2 unknowns per element.  The
operator is assembled here on the device, from the seed: base state phases,
then a normally distributed solution x* with right-hand side b = A x* (and
lambda* with g = A^T lambda* for the adjoint), so that the exact answer of a
solve is known without solving.

Kinds:
    spmv      y = A x or A^T x
    apply     M^-1 r or M^-T r with a factorization that the program keeps
    system    factor A and solve A x = b
    refactor  new values in an old pattern (the next pseudo-time step): refactor, solve
    gradient  x = A^-1 b and its gradients with respect to A's values and b
    batch     factor and solve several systems of different sizes together
"""
import math

import numpy as np
import torch

import paper_2101_01763_amd as sp

GAMMA = 1.4


# ------------------------------------------------------------------ cases

def listed():
    return [
        # The smallest call of the library: one operator product of the 16x16,
        # p = 1 test grid.  Launch and call latency.
        dict(name="spmv_small", kind="spmv", nx=16, ny=16, p=1, py=False, transpose=False),
        # The operator of an adjoint solve at the benchmark's grid: bandwidth.
        dict(name="spmv_t_large", kind="spmv", nx=256, ny=256, p=3, py=False, transpose=True),
        # A preconditioner that a Krylov method of the user's own applies in
        # full precision, on the 128x128, p = 2 grid of the tests.
        dict(name="apply_f64", kind="apply", nx=128, ny=128, p=2, py=False, eps=1e-2, dtype="f64", transpose=False),
        # The transposed one on a small odd grid, periodic both ways: the sweep's latency.
        dict(name="apply_t_small_f64", kind="apply", nx=37, ny=29, p=1, py=True, eps=1e-2, dtype="f64", transpose=True),
        # The smallest whole call: the 16x16, p = 1 system, solved with the s and
        # restart that the benchmark uses for it.
        dict(name="system_small_f64", kind="system", nx=16, ny=16, p=1, py=False, eps=1e-2, dtype="f64", s=4, restart=40,
             lagged=False),
        # An ordinary one, on an odd grid that does not divide into even boxes, FP64 factor.
        dict(name="system_ragged_f64", kind="system", nx=91, ny=69, p=3, py=False, eps=1e-2, dtype="f64", s=5, restart=60,
             lagged=False),
        # The 128x128, p = 2 system with the FP32 factor, default schedule.
        dict(name="system_mid_f32", kind="system", nx=128, ny=128, p=2, py=False, eps=1e-2, dtype="f32", s=5, restart=60,
             lagged=False),
        # A p = 1 operator: small blocks, few iterations, at the loose tolerance.
        dict(name="system_p1_f32", kind="system", nx=160, ny=120, p=1, py=False, eps=1e-1, dtype="f32", s=5, restart=60,
             lagged=True),
        # The benchmark's workload: 256x256, p = 3, FP32 factor, single-reduce schedule.
        dict(name="system_large_f32", kind="system", nx=256, ny=256, p=3, py=False, eps=1e-2, dtype="f32", s=5, restart=60,
             lagged=True),
        # The next step of a pseudo-transient loop: new values, tighter tolerance.
        dict(name="refactor_f32", kind="refactor", nx=96, ny=96, p=2, py=False, eps=1e-3, dtype="f32", s=5, restart=60,
             lagged=True),
        # Gradients of a solve at 192x192, p = 2 with a factorization in hand:
        # forward solve, adjoint solve, pattern outer product.
        dict(name="gradient_f32", kind="gradient", nx=192, ny=192, p=2, py=False, eps=1e-2, dtype="f32", s=5, restart=60,
             lagged=False),
        # Ten systems of a parameter study: grids of 32 to 96 elements a side, p = 1 to 3.
        dict(name="batch_f32", kind="batch", count=10, p=0, lo=32, hi=96, eps=1e-2, dtype="f32", s=5, restart=60, lagged=True,
             sizes=7),
    ]


def draw(rng):
    kind = rng.choice(["spmv", "apply", "system", "system", "refactor", "gradient", "batch"])
    if kind == "batch":
        p, dtype = rng.choice([0, 1, 2, 3]), rng.choice(["f32", "f32", "f64"])
        most = (12 if p in (0, 1) else 8) // (2 if dtype == "f64" else 1)  # at most the largest listed case's work
        return dict(kind=kind, count=rng.randint(2, most), p=p, lo=rng.randint(16, 40), hi=rng.randint(48, 80),
                    eps=rng.choice([1e-1, 1e-2]), dtype=dtype, s=5, restart=60, lagged=rng.random() < 0.5,
                    sizes=rng.randint(0, 1 << 20))
    p = rng.randint(1, 3)
    b = 4 * (p + 1) ** 2
    dtype = "f64" if kind == "apply" else rng.choice(["f32", "f64"])
    # unknowns, log-uniform up to the largest listed case of the kind
    top = {"spmv": 4.1e6, "apply": 6e5, "system": 1.5e6 if dtype == "f32" else 6e5, "refactor": 3.3e5, "gradient": 6e5}[kind]
    bottom = 4096.0 if kind != "gradient" else 2e4
    n = math.exp(rng.uniform(math.log(bottom), math.log(top)))
    aspect = math.exp(rng.uniform(math.log(0.5), math.log(2.0)))
    c = dict(kind=kind, nx=max(6, min(256, int(round(math.sqrt(n / b * aspect))))),
             ny=max(6, min(256, int(round(math.sqrt(n / b / aspect))))), p=p, py=rng.random() < 0.25)
    if kind in ("spmv", "apply"):
        c["transpose"] = rng.random() < 0.5
    if kind == "apply":
        c.update(eps=rng.choice([1e-1, 1e-2, 1e-3]), dtype=dtype)
    if kind not in ("spmv", "apply"):
        c.update(eps=1e-3 if kind == "refactor" else rng.choice([1e-1, 1e-2]), dtype=dtype, s=rng.choice([4, 5, 5]), restart=60,
                 lagged=kind != "gradient" and rng.random() < 0.5)
    return c


# --------------------------------------------------------------- operator

def _flux_jacobians(U):
    rho, u, v = U[:, 0], U[:, 1] / U[:, 0], U[:, 2] / U[:, 0]
    q2, g1 = u * u + v * v, GAMMA - 1.0
    pr = g1 * (U[:, 3] - 0.5 * rho * q2)
    H = (U[:, 3] + pr) / rho
    z, o = torch.zeros_like(rho), torch.ones_like(rho)
    A = [[z, o, z, z], [0.5 * g1 * q2 - u * u, (3 - GAMMA) * u, -g1 * v, g1 * o], [-u * v, v, u, z],
         [u * (0.5 * g1 * q2 - H), H - g1 * u * u, -g1 * u * v, GAMMA * u]]
    B = [[z, z, o, z], [-u * v, v, u, z], [0.5 * g1 * q2 - v * v, -g1 * u, (3 - GAMMA) * v, g1 * o],
         [v * (0.5 * g1 * q2 - H), -g1 * u * v, H - g1 * v * v, GAMMA * v]]
    c = torch.sqrt(GAMMA * pr / rho)
    mat = lambda M: torch.stack([torch.stack(r, -1) for r in M], -2)  # noqa: E731
    return mat(A), mat(B), u, v, c


def _conserved(rho, u, v, pr):
    return torch.stack([rho, rho * u, rho * v, pr / (GAMMA - 1.0) + 0.5 * rho * (u * u + v * v)], -1)


class Operator:
    """The Jacobian of an nx x ny grid at order p about a seeded base state."""

    def __init__(self, nx, ny, p, py, gen, mach=0.5, alpha=2.0, cfl=10.0, dev="cuda"):
        q, K = p + 1, nx * ny
        self.nx, self.ny, self.b, self.K, self.N, self.py = nx, ny, 4 * q * q, K, 4 * q * q * K, py
        f8 = dict(dtype=torch.float64, device=dev)
        e = np.arange(K)
        i, j = e % nx, e // nx
        right, left = j * nx + (i + 1) % nx, j * nx + (i - 1) % nx
        top, bot = ((j + 1) % ny) * nx + i, ((j - 1) % ny) * nx + i
        if not py:
            top, bot = np.where(j == ny - 1, -1, top), np.where(j == 0, -1, bot)
        nbrs = [e, right, left, top, bot]
        rows = np.concatenate([e[n >= 0] for n in nbrs])
        cols = np.concatenate([n[n >= 0] for n in nbrs])
        order = np.argsort(rows * np.int64(K) + cols, kind="stable")
        place = np.empty(len(order), np.int64)
        place[order] = np.arange(len(order))
        slots, off = [], 0
        for n in nbrs:  # block number of each element's coupling to that neighbour, -1 where there is none
            s = np.full(K, -1, np.int64)
            s[n >= 0] = place[off:off + int((n >= 0).sum())]
            off += int((n >= 0).sum())
            slots.append(s)
        dv = lambda a: torch.as_tensor(a, device=dev)  # noqa: E731
        self.rowptr = dv(np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=K))]).astype(np.int32))
        self.colind = dv(cols[order].astype(np.int32))
        # (elements, their neighbours, block numbers) of each of the five couplings
        self.parts = [(dv(e[n >= 0]), dv(n[n >= 0]), dv(s[n >= 0])) for n, s in zip(nbrs, slots)]

        ph = 2 * math.pi * torch.rand(8, generator=gen, **f8)
        a = math.radians(alpha)
        winf = [1.0, math.cos(a), math.sin(a), 1.0 / (GAMMA * mach * mach)]
        X, Y = dv((i + 0.5) / nx), dv((j + 0.5) / ny)
        w = [winf[k] * (1.0 + 0.05 * torch.sin(2 * math.pi * X + ph[k]) * torch.sin(2 * math.pi * Y + ph[4 + k])) for k in range(4)]
        U = _conserved(*w)
        Uinf = _conserved(*[torch.full((1,), t, **f8) for t in winf])
        Ax, By, u, v, c = _flux_jacobians(U)
        _, _, ui, vi, ci = _flux_jacobians(Uinf)
        h = 1.0 / max(nx, ny)
        hh = 0.5 * h
        I, I4 = np.eye(q), torch.eye(4, **f8)
        S = np.zeros((q, q))
        for m in range(q):
            for k in range(m):
                if (m + k) % 2:
                    S[k, m] = math.sqrt((2 * m + 1) * (2 * k + 1))
        P = np.sqrt((2 * np.arange(q) + 1) / 2.0)
        Q = P * (-1.0) ** np.arange(q)
        val = torch.zeros(len(order), self.b, self.b, **f8)

        def add(slot, modes, flux):  # val[slot] += modes (x) flux
            m = dv(modes).view(1, q * q, 1, q * q, 1) * flux.view(-1, 1, 4, 1, 4)
            val[slot] += m.view(-1, self.b, self.b)

        diag = self.parts[0][2]
        add(diag, np.kron(S.T, I), -hh * Ax)
        add(diag, np.kron(I, S.T), -hh * By)
        for k, (sgn, Jac, vel, veli, t, o, inx) in enumerate([(1.0, Ax, u, ui, P, Q, True), (-1.0, Ax, u, ui, Q, P, True),
                                                              (1.0, By, v, vi, P, Q, False), (-1.0, By, v, vi, Q, P, False)]):
            el, nb, slot = self.parts[k + 1]
            own = torch.abs(vel) + c
            other = (torch.abs(veli) + ci).expand(K).clone()
            other[el] = own[nb]
            lam = torch.maximum(own, other).view(-1, 1, 1)
            kk, kn = np.outer(t, t), np.outer(t, o)
            add(diag, np.kron(kk, I) if inx else np.kron(I, kk), hh * (0.5 * sgn * Jac + 0.5 * lam * I4))
            add(slot, np.kron(kn, I) if inx else np.kron(I, kn), hh * (0.5 * sgn * Jac[nb] - 0.5 * lam[el] * I4))
        dtau = cfl / ((2 * p + 1) * (torch.sqrt(u * u + v * v) + c) / h).max()
        val.diagonal(dim1=1, dim2=2)[diag] += hh * hh / dtau
        self.val = val

    def times(self, x):
        """A x, block by block in torch."""
        y, xb = torch.zeros(self.K, self.b, 1, dtype=torch.float64, device=x.device), x.view(self.K, self.b, 1)
        for el, nb, slot in self.parts:
            y[el] += torch.bmm(self.val[slot], xb[nb])
        return y.view(-1)

    def t_times(self, x):
        """A^T x, block by block in torch."""
        y, xb = torch.zeros(self.K, 1, self.b, dtype=torch.float64, device=x.device), x.view(self.K, 1, self.b)
        for el, nb, slot in self.parts:
            y[nb] += torch.bmm(xb[el], self.val[slot])
        return y.view(-1)

    def matrix(self):
        return sp.BSRMatrix(self.rowptr, self.colind, self.val)


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 7919 + 1)
    return g


def _normal(n, gen):
    return torch.randn(n, generator=gen, dtype=torch.float64, device="cuda")


def _made(case, seed):
    """The operator of a case and its generator, at the point where x* is drawn."""
    gen = _generator(seed)
    return Operator(case["nx"], case["ny"], case["p"], case["py"], gen), gen


def _batch_grids(case):
    """Grid sides, orders, Mach numbers and angles of a batch: of the case, not of the seed."""
    r = np.random.default_rng(case["sizes"])
    return [(int(r.integers(case["lo"], case["hi"] + 1)), case["p"] or int(r.integers(1, 4)), float(r.uniform(0.3, 0.7)),
             float(r.uniform(-4.0, 4.0))) for _ in range(case["count"])]


def _batch(case, seed):
    gen = _generator(seed)
    out = []
    for n, p, mach, alpha in _batch_grids(case):
        A = Operator(n, n, p, False, gen, mach=mach, alpha=alpha)
        out.append((A, _normal(A.N, gen)))
    return out


# ---------------------------------------------------------------- the run

def _factor(A, case):
    return sp.factor(A.matrix(), A.nx, A.ny, True, A.py, eps=case["eps"], nlevels=sp.levels_for(A.N), dtype=case["dtype"])


def prepare(case, seed):
    kind, st = case["kind"], dict(case=case)
    if kind == "batch":
        made = _batch(case, seed)
        st["systems"] = [(A.matrix(), A.nx, A.ny, True, False) for A, _ in made]
        st["levels"] = [sp.levels_for(A.N) for A, _ in made]
        st["b"] = [A.times(x) for A, x in made]
        return st
    A, gen = _made(case, seed)
    st.update(op=A, A=A.matrix())
    if kind == "spmv":
        st["x"] = _normal(A.N, gen)
    elif kind == "apply":
        st["M"] = _factor(A, case)
        st["x"] = _normal(A.N, gen)
    else:
        st["b"] = A.times(_normal(A.N, gen))
    if kind == "gradient":
        st["M"] = _factor(A, case)
        st["g"] = A.t_times(_normal(A.N, gen))
        st["vals"] = A.val.clone().requires_grad_()
        st["b"].requires_grad_()
    if kind == "refactor":  # the factorization of the step before: another base state in the same pattern
        st["M"] = _factor(_made(case, seed + (1 << 20))[0], case)
    return st


def run(st):
    case, kind = st["case"], st["case"]["kind"]
    if kind == "spmv":
        return sp.spmv(st["A"], st["x"], transpose=case["transpose"])
    if kind == "apply":
        return st["M"].apply_T(st["x"]) if case["transpose"] else st["M"].apply(st["x"])
    how = dict(s=case["s"], restart=case["restart"], rtol=1e-8)
    if kind == "system":
        M = _factor(st["op"], case)
        x, _ = sp.solve(st["A"], st["b"], M, lagged=case["lagged"], **how)
        return x
    if kind == "refactor":
        st["M"].refactor(st["A"])
        x, _ = sp.solve(st["A"], st["b"], st["M"], lagged=case["lagged"], **how)
        return x
    if kind == "gradient":
        x = sp.SpandSolve.apply(st["vals"], st["b"], st["A"], st["M"], how)
        dvals, db = torch.autograd.grad(x, [st["vals"], st["b"]], st["g"])
        return dict(x=x.detach(), dvals=dvals, db=db)
    Ms = sp.factor_batched(st["systems"], eps=case["eps"], nlevels=st["levels"], dtype=case["dtype"])
    xs, _ = sp.solve_batched([s[0] for s in st["systems"]], st["b"], Ms, lagged=case["lagged"], **how)
    return xs


# ------------------------------------------------------- floors and answers

def _work_of(nx, ny, p, py, case):
    """Bytes and operations of one system: the operator and the vectors once,
    and the inversion of the leaves (their blocks read once, for an apply)."""
    b, K = 4 * (p + 1) ** 2, nx * ny
    N, nnzb = K * b, 5 * K - (0 if py else 2 * nx)
    mat, vec = 8.0 * nnzb * b * b + 4.0 * nnzb + 4.0 * (K + 1), 16.0 * N
    if case["kind"] == "spmv":
        return mat + vec, 2.0 * nnzb * b * b
    boxes = 2.0 ** (sp.levels_for(N) - 1)
    m = max(1.0, (math.sqrt(K / boxes) - 1.0) ** 2) * b  # unknowns of a leaf without its separators
    if case["kind"] == "apply":
        return boxes * m * m * (8 if case["dtype"] == "f64" else 4) + vec, 2.0 * boxes * m * m
    leaves = 2.0 * boxes * m ** 3
    if case["kind"] == "gradient":
        return 2 * mat + 4 * vec, 4.0 * boxes * m * m + 3.0 * nnzb * b * b
    return mat + vec, leaves


def work(case):
    if case["kind"] == "batch":
        w = [_work_of(n, n, p, False, case) for n, p, _, _ in _batch_grids(case)]
    else:
        w = [_work_of(case["nx"], case["ny"], case["p"], case["py"], case)]
    return {"bytes": sum(t[0] for t in w), "flops": sum(t[1] for t in w)}


def exact(case, seed):
    """The solution that the right-hand side was made from (in 64 bits); a
    preconditioner at a tolerance has no such value."""
    kind = case["kind"]
    if kind == "apply":
        return None
    if kind == "batch":
        return [x for _, x in _batch(case, seed)]
    A, gen = _made(case, seed)
    x = _normal(A.N, gen)
    if kind == "spmv":
        return A.t_times(x) if case["transpose"] else A.times(x)
    if kind != "gradient":
        return x
    lam = _normal(A.N, gen)
    dvals = torch.empty_like(A.val)
    for el, nb, slot in A.parts:
        dvals[slot] = -lam.view(A.K, A.b, 1)[el] * x.view(A.K, 1, A.b)[nb]
    return dict(x=x, dvals=dvals, db=lam)
