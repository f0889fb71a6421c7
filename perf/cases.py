"""Performance cases of the bake-off library through its public entry points.

A case is one call (or one short group of calls) that a user's program makes
in earnest: a Jacobi-PCG solve, one application of an assembled or
element-local operator, the mixed-precision solve, or the coefficient part of
a step of the inverse problem. `prepare` builds what such a program holds
beforehand (the mesh's operator and the device vectors), `run` makes the call,
`work` counts the bytes and operations it cannot do without, and `exact`
states the same result in plain FP64 torch, without the library.
"""
from __future__ import annotations

import math

import numpy as np
import torch

# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

_DEFAULTS = {"bp": 5, "p": 7, "ex": 4, "ey": 4, "ez": 4, "ncomp": 1, "iters": 20, "beta": 0.0,
             "fp32": False, "random_map": False, "caller_order": False}


def _case(kind, **kw):
    return {"kind": kind, **_DEFAULTS, **kw}


def listed():
    """The listed cases: each of the calls above, from the smallest sizes to the largest."""
    return [
        # a small problem, as each rank of a strongly scaled run or a coarse
        # level holds it: launches and latency count, not bandwidth
        _case("solve", name="bp5_solve_small", ex=4, ey=4, ez=2, iters=60),
        # the size at which a GPU first reaches most of its rate (n_0.8)
        _case("solve", name="bp5_solve_mid", ex=16, ey=16, ez=8, iters=60),
        # the headline benchmark: scalar Poisson, collocated GLL points
        _case("solve", name="bp5_solve_large", ex=64, ey=64, ez=64, iters=20),
        # scalar Poisson with over-integration (Gauss points)
        _case("solve", name="bp3_solve_large", bp=3, ex=48, ey=48, ez=48, iters=20),
        # mass matrix solve (projection onto the space), uneven element counts,
        # the mesh's own lexicographic numbering kept as its benchmark does
        _case("solve", name="bp1_solve_ragged", bp=1, p=6, ex=41, ey=37, ez=29, iters=20,
              caller_order=True),
        # vector Poisson, three components on one mesh
        _case("solve", name="bp6_solve_vector", bp=6, ex=32, ey=32, ez=32, ncomp=3, iters=20),
        # an implicit viscous step of a three-component velocity: Helmholtz
        # with Gauss points on an unstructured numbering, solved to tolerance
        _case("helmholtz", name="helmholtz_step", bp=4, p=5, ex=17, ey=13, ez=11, ncomp=3,
              beta=2000.0, random_map=True),
        # one small operator application, as another library's Krylov loop makes it
        _case("apply", name="apply_small", p=5, ex=6, ey=5, ez=4),
        # one large application at a high order
        _case("apply", name="apply_large", p=8, ex=40, ey=36, ez=33),
        # the unassembled element kernel at an order above the usual range
        _case("local", name="local_high_order", p=11, ex=20, ey=18, ez=17),
        # FP32 inner iterations with FP64 corrections, to the default tolerance
        _case("mixed", name="mixed_solve", ex=16, ey=16, ez=16, fp32=True),
        # the inverse problem's work around its solves: a new coefficient, the
        # preconditioner's diagonal, the misfit and the coefficient gradient
        _case("adjoint", name="adjoint_step", p=5, ex=32, ey=32, ez=32, ncomp=8),
    ]


def _grid(rng, p, lo, hi):
    """Uneven element counts whose node count is log-uniform in [lo, hi]."""
    n = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    m = max(1.0, (n / p ** 3) ** (1.0 / 3.0))
    ex, ey = (max(1, round(m * math.exp(rng.uniform(-0.3, 0.3)))) for _ in range(2))
    ez = max(1, round(n / p ** 3 / (ex * ey)))
    return ex, ey, ez


def draw(rng):
    """One more case of the ranges that the listed ones stand for."""
    kind = rng.choice(["solve", "solve", "solve", "solve", "apply", "apply", "local", "helmholtz",
                       "mixed", "adjoint"])
    c = _case(kind)
    c["random_map"] = rng.random() < 0.2
    if kind == "solve":
        c["bp"] = rng.choice([1, 2, 3, 4, 5, 5, 6])
        c["p"] = rng.choice([1, 2, 3, 4, 5, 6, 7, 7, 8] if c["bp"] < 5 else
                            [2, 3, 4, 5, 6, 7, 7, 7, 8, 9, 11])
        c["ncomp"] = 3 if c["bp"] in (2, 4, 6) else 1
        c["iters"] = rng.randint(20, 60)
        c["caller_order"] = c["bp"] <= 2 and not c["random_map"]
        lo, hi = 1e4, 2e7 / c["ncomp"]
    elif kind == "apply":
        c["bp"] = rng.choice([1, 3, 5, 5, 6])
        c["p"] = rng.randint(2, 8 if c["bp"] < 5 else 12)
        c["ncomp"] = 3 if c["bp"] == 6 else 1
        c["fp32"] = rng.random() < 0.4
        lo, hi = 5e3, 3e7 / c["ncomp"]
    elif kind == "local":
        c["bp"] = rng.choice([1, 3, 5, 5, 5])
        c["p"] = rng.randint(2, 8 if c["bp"] < 5 else 15)
        c["fp32"] = rng.random() < 0.3
        c["random_map"] = False
        lo, hi = 1e4, 3e7
    elif kind == "helmholtz":
        c["bp"] = rng.choice([3, 4, 5, 6])
        c["p"] = rng.randint(3, 8)
        c["ncomp"] = 3 if c["bp"] in (4, 6) else 1
        c["beta"] = math.exp(rng.uniform(math.log(500.0), math.log(8000.0)))
        lo, hi = 1e4, 1.5e6 / c["ncomp"]
    elif kind == "mixed":
        c["p"] = rng.randint(4, 8)
        c["fp32"] = True
        lo, hi = 3e4, 2e6
    else:
        c["p"] = rng.randint(3, 7)
        c["ncomp"] = rng.randint(1, 8)
        lo, hi = 2e4, 2e7 / c["ncomp"]
    c["ex"], c["ey"], c["ez"] = _grid(rng, c["p"], lo, hi)
    return c


# ---------------------------------------------------------------------------
# one-dimensional rules (for the meshes and the FP64 statement)
# ---------------------------------------------------------------------------

def _legendre(n, x):
    """P_n, P_n' and P_{n-1} at x."""
    a, b = np.ones_like(x), np.array(x, dtype=np.float64)
    for k in range(2, n + 1):
        a, b = b, ((2 * k - 1) * x * b - (k - 1) * a) / k
    return b, n * (x * b - a) / (x * x - 1.0), a


def _gll(n):
    """GLL points and weights: the ends and the roots of P'_{n-1}."""
    m = n - 1
    x = -np.cos(np.pi * np.arange(n) / m)
    for _ in range(50):
        pm, dpm, _ = _legendre(m, x[1:-1])
        d2 = (2.0 * x[1:-1] * dpm - m * (m + 1) * pm) / (1.0 - x[1:-1] ** 2)
        x[1:-1] -= dpm / d2
    x = 0.5 * (x - x[::-1])
    a, b = np.ones_like(x), x.copy()
    for k in range(2, m + 1):
        a, b = b, ((2 * k - 1) * x * b - (k - 1) * a) / k
    return x, 2.0 / (m * n * b * b)


def _lagrange(nodes, pts):
    """(J, D): the nodes' Lagrange polynomials and their derivatives at pts."""
    n = nodes.size
    J = np.ones((pts.size, n))
    D = np.zeros((pts.size, n))
    for i in range(n):
        others = [m for m in range(n) if m != i]
        for m in others:
            J[:, i] *= (pts - nodes[m]) / (nodes[i] - nodes[m])
        for s in others:
            term = np.full(pts.size, 1.0 / (nodes[i] - nodes[s]))
            for m in others:
                if m != s:
                    term *= (pts - nodes[m]) / (nodes[i] - nodes[m])
            D[:, i] += term
    return J, D


def _gauss(case):
    """Whether the case's problem uses Gauss points (BP1-BP4)."""
    return case["bp"] <= 4


def _points(case):
    return case["p"] + (2 if _gauss(case) else 1)


def _nodes_total(case):
    p = case["p"]
    return (p * case["ex"] + 1) * (p * case["ey"] + 1) * (p * case["ez"] + 1)


# ---------------------------------------------------------------------------
# inputs, made on the device from the seed
# ---------------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _mesh(case, seed, xi):
    """Map [E, p1^3], coordinates [E, p1^3, 3] and boundary flags [n] (device)
    of a brick of trilinear elements whose vertices are moved by a smooth map."""
    p, ex, ey, ez = case["p"], case["ex"], case["ey"], case["ez"]
    p1 = p + 1
    f64 = {"dtype": torch.float64, "device": "cuda"}
    rng = np.random.default_rng(int(seed))
    axes = [torch.linspace(0.0, 1.0, m + 1, **f64) for m in (ez, ey, ex)]
    Z, Y, X = torch.meshgrid(*axes, indexing="ij")
    h, bump = 1.0 / max(ex, ey, ez), (torch.sin(math.pi * X) * torch.sin(math.pi * Y)
                                      * torch.sin(math.pi * Z))
    k, phase = rng.integers(1, 3, size=(3, 3)), rng.uniform(0.0, 2.0 * math.pi, size=3)
    V = torch.stack([v + 0.1 * h * bump * torch.sin(2.0 * math.pi * (int(k[c, 0]) * X
                     + int(k[c, 1]) * Y + int(k[c, 2]) * Z) + float(phase[c]))
                     for c, v in enumerate((X, Y, Z))])            # [3, ez+1, ey+1, ex+1]
    corners = torch.stack([V[:, cz:cz + ez, cy:cy + ey, cx:cx + ex].reshape(3, -1)
                           for cz in (0, 1) for cy in (0, 1) for cx in (0, 1)], dim=2)
    lin = np.stack([(1.0 - xi) / 2, (1.0 + xi) / 2], axis=1)
    W = np.einsum("kc,jb,ia->kjicba", lin, lin, lin).reshape(p1 ** 3, 8)
    E = ex * ey * ez
    xyz = corners.reshape(3 * E, 8) @ torch.tensor(W.T.copy(), **f64)
    xyz = xyz.reshape(3, E, p1 ** 3).permute(1, 2, 0).contiguous()
    nx, ny, nz = p * ex + 1, p * ey + 1, p * ez + 1
    e = torch.arange(E, device="cuda")
    base = p * (e % ex) + nx * p * (e // ex % ey) + nx * ny * p * (e // (ex * ey))
    l = torch.arange(p1 ** 3, device="cuda")
    dofs = base[:, None] + (l % p1 + nx * (l // p1 % p1) + nx * ny * (l // (p1 * p1)))[None, :]
    g = torch.arange(nx * ny * nz, device="cuda")
    gi, gj, gk = g % nx, g // nx % ny, g // (nx * ny)
    boundary = ((gi == 0) | (gi == nx - 1) | (gj == 0) | (gj == ny - 1) | (gk == 0)
                | (gk == nz - 1)).to(torch.uint8)
    if case["random_map"]:  # arbitrary node ids and element order
        gen = _generator(seed)
        new = torch.randperm(g.numel(), generator=gen, device="cuda")
        order = torch.randperm(E, generator=gen, device="cuda")
        dofs, xyz = new[dofs[order]], xyz[order]
        boundary = torch.empty_like(boundary).index_copy_(0, new, boundary)
    return dofs, xyz, boundary


def _dirichlet(case):
    return case["bp"] >= 3


def _uniform(gen, *shape):
    return torch.rand(*shape, generator=gen, dtype=torch.float64, device="cuda") * 2.0 - 1.0


def _vectors(case, seed, xyz, dofs, boundary):
    """The device vectors of the call."""
    gen = _generator(int(seed) + 7919)
    n, nc, kind = _nodes_total(case), case["ncomp"], case["kind"]
    free = 1.0 - boundary.double() if _dirichlet(case) else torch.ones(n, dtype=torch.float64,
                                                                       device="cuda")
    shape = (n,) if nc == 1 else (nc, n)
    if kind == "local":
        t = _uniform(gen, nc, dofs.shape[0], (case["p"] + 1) ** 3)
        return {"u": t.float() if case["fp32"] else t}
    if kind == "apply":
        t = _uniform(gen, *shape)
        return {"u": t.float() if case["fp32"] else t}
    if kind == "mixed":  # f at the nodes, seeded modes of the sine basis; b = M f
        at = torch.empty(n, 3, dtype=torch.float64, device="cuda")
        at[dofs.reshape(-1)] = xyz.reshape(-1, 3)
        amp = _uniform(gen, 3, 3)
        return {"f": sum(amp[i, j] * torch.sin(math.pi * (i + 1) * at[:, 0])
                         * torch.sin(math.pi * (j + 1) * at[:, 1]) * torch.sin(math.pi * at[:, 2])
                         for i in range(3) for j in range(3)) * free}
    if kind == "adjoint":
        q3 = _points(case) ** 3
        return {"kappa": torch.exp(0.5 * _uniform(gen, dofs.shape[0], q3)),
                "u": _uniform(gen, *shape), "target": _uniform(gen, *shape),
                "lam": _uniform(gen, *shape)}
    return {"b": _uniform(gen, *shape) * free}


def prepare(case, seed):
    """The operator on the case's mesh and the vectors, as a program holds them."""
    from paper_2004_06722_amd import bp

    xi, _ = bp.rule(case["p"] + 1, bp.GLL)
    dofs, xyz, boundary = _mesh(case, seed, xi)
    q, quad = bp.bp_quadrature(case["bp"], case["p"])
    op = bp.Operator(case["p"], q, quad, dofs.cpu().numpy(), xyz.cpu().numpy(),
                     _nodes_total(case),
                     dirichlet=boundary.cpu().numpy() if _dirichlet(case) else None,
                     ncomp=case["ncomp"], fp32=case["fp32"], caller_order=case["caller_order"])
    if case["kind"] == "helmholtz":
        op.set_helmholtz(case["beta"])
    state = {"case": case, "op": op, **_vectors(case, seed, xyz, dofs, boundary)}
    if case["kind"] == "mixed":
        state["b"] = op.apply(bp.MASS, state.pop("f"))
    return state


def _which(case):
    return {"helmholtz": "HELM"}.get(case["kind"], "MASS" if case["bp"] <= 2 else "STIFF")


def run(state):
    """One pass: the call itself, as a user's program makes it."""
    from paper_2004_06722_amd import bp

    case, op = state["case"], state["op"]
    which, kind = getattr(bp, _which(case)), case["kind"]
    if kind == "solve":
        x, st = op.pcg_solve(state["b"], which=which, maxit=case["iters"], fixed_iters=True)
        return {"x": x, "rel_res": st["rel_res"][0], "iters": st["iters"]}
    if kind == "helmholtz":  # rounding may move the last iteration: the solution alone
        return {"x": op.pcg_solve(state["b"], which=which, rtol=1e-12)[0]}
    if kind == "mixed":
        return {"x": op.pcg_solve_mixed(state["b"])[0]}
    if kind == "apply":
        return {"w": op.apply(which, state["u"])}
    if kind == "local":
        return {"w": op.apply_local(which, state["u"])}
    op.set_coeff(state["kappa"])
    diag = op.diag(bp.STIFF)
    loss, grad = op.mass_misfit(state["u"], state["target"])
    return {"diag": diag, "loss": loss, "grad": grad,
            "grad_kappa": op.grad_kappa(state["lam"], state["u"])}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _element_flops(case, stiff=True):
    """Operations of one element's operator by sum factorisation."""
    p1, q = case["p"] + 1, _points(case)
    if not _gauss(case):
        return 12 * p1 ** 4 + 15 * p1 ** 3 if stiff else p1 ** 3
    interp = 4 * (p1 ** 3 * q + p1 ** 2 * q ** 2 + p1 * q ** 3)
    return interp + (12 * q ** 4 + 15 * q ** 3 if stiff else q ** 3)


def work(case):
    """Bytes and operations of one pass: inputs read and outputs written once
    per operator application, the iteration's vectors once per iteration."""
    E, p1, q = case["ex"] * case["ey"] * case["ez"], case["p"] + 1, _points(case)
    n, nc, kind = _nodes_total(case), case["ncomp"], case["kind"]
    word = 4 if case["fp32"] else 8
    stiff = _which(case) != "MASS"
    data = E * q ** 3 * ((6 if stiff else 1) + (1 if kind == "helmholtz" else 0))
    if kind == "local":
        return {"bytes": word * (data + 2 * nc * E * p1 ** 3),
                "flops": nc * E * _element_flops(case, stiff)}
    if kind == "apply":
        return {"bytes": word * (data + 2 * nc * n) + 4 * E * p1 ** 3,
                "flops": nc * E * _element_flops(case, stiff)}
    if kind == "adjoint":
        # kappa and G in, kappa G out; kappa G, map and diagonal; B~, map, u,
        # target and gradient; G, map, lam, u and the coefficient gradient
        q3 = E * q ** 3
        return {"bytes": 8 * (13 * q3 + 6 * q3 + n + q3 + 3 * nc * n + 6 * q3 + 2 * nc * n + q3)
                + 3 * 4 * E * p1 ** 3,
                "flops": nc * E * (_element_flops(case) * 2 + 3 * q ** 3)}
    # an iteration: the operator's data and map, u and w, and x, p, z in and
    # out with w and the preconditioner in; the tolerance modes by a typical count
    iters = {"helmholtz": 80, "mixed": 600}.get(kind, case["iters"])
    vec = (2 + 7) * nc * n + n
    return {"bytes": iters * (word * (data + vec) + 4 * E * p1 ** 3),
            "flops": iters * nc * (E * _element_flops(case, stiff) + 12 * n)}


# ---------------------------------------------------------------------------
# the same results in plain FP64 torch
# ---------------------------------------------------------------------------

class _Plain:
    """The discretisation stated directly: geometric factors at the points,
    tensor contractions by matrix products, gather and scatter by index."""

    def __init__(self, case, seed):
        p1, q = case["p"] + 1, _points(case)
        xi, wi = _gll(p1)
        eta, rho = np.polynomial.legendre.leggauss(q) if _gauss(case) else (xi, wi)
        dofs, xyz, boundary = _mesh(case, seed, xi)
        self.vectors = _vectors(case, seed, xyz, dofs, boundary)
        f64 = {"dtype": torch.float64, "device": "cuda"}
        J, D = _lagrange(xi, eta)
        self.J, self.D = torch.tensor(J, **f64), torch.tensor(D, **f64)
        self.colloc = not _gauss(case)
        self.p1, self.q, self.E, self.n = p1, q, dofs.shape[0], boundary.numel()
        self.map = dofs.reshape(-1)
        self.free = 1.0 - boundary.double() if _dirichlet(case) else None
        M = [[None] * 3 for _ in range(3)]
        for l in range(3):
            X = xyz[:, :, l].reshape(self.E, p1, p1, p1).contiguous()
            for m, d in enumerate(self.gradient(X)):
                M[l][m] = d
        del xyz
        cof = [[M[(l + 1) % 3][(m + 1) % 3] * M[(l + 2) % 3][(m + 2) % 3]
                - M[(l + 1) % 3][(m + 2) % 3] * M[(l + 2) % 3][(m + 1) % 3] for m in range(3)]
               for l in range(3)]
        det = sum(M[0][m] * cof[0][m] for m in range(3))
        del M
        r = torch.tensor(rho, **f64)
        w = r[:, None, None] * r[None, :, None] * r[None, None, :]
        self.B = det * w
        self.G = {}
        if case["bp"] >= 3 or case["kind"] == "adjoint":
            for a in range(3):
                for b in range(a, 3):
                    self.G[a, b] = sum(cof[l][a] * cof[l][b] for l in range(3)) * (w / det)

    @staticmethod
    def along(x, A, d):
        """Contract direction d (0 fastest) of x [E, k, j, i] with A [out, in]."""
        y = x.transpose(3 - d, 3)
        y = (y.reshape(-1, y.shape[3]) @ A.T).reshape(*y.shape[:3], A.shape[0])
        return y.transpose(3 - d, 3).contiguous()

    def tensor(self, x, mats):
        for d, A in enumerate(mats):
            if A is not None:
                x = self.along(x, A, d)
        return x

    def gradient(self, x):
        J = None if self.colloc else self.J
        return [self.tensor(x, [self.D if d == m else J for d in range(3)]) for m in range(3)]

    def g(self, a, b):
        return self.G[min(a, b), max(a, b)]

    def stiff_local(self, x, kappa=None):
        d = self.gradient(x)
        Jt = None if self.colloc else self.J.T.contiguous()
        Dt = self.D.T.contiguous()
        out = torch.zeros_like(x)
        for a in range(3):
            v = sum(self.g(a, b) * d[b] for b in range(3))
            v = v if kappa is None else kappa * v
            out += self.tensor(v, [Dt if c == a else Jt for c in range(3)])
        return out

    def mass_local(self, x):
        if self.colloc:
            return self.B * x
        v = self.B * self.tensor(x, [self.J] * 3)
        return self.tensor(v, [self.J.T.contiguous()] * 3)

    def gather(self, u):
        return u[self.map].reshape(self.E, self.p1, self.p1, self.p1)

    def scatter(self, xl):
        return torch.zeros(self.n, dtype=torch.float64, device="cuda").index_add_(
            0, self.map, xl.reshape(-1))

    def operator(self, which, beta=0.0, masked=True):
        mask = self.free if masked and self.free is not None else None

        def apply(u):
            x = self.gather(u if mask is None else u * mask)
            y = self.mass_local(x) if which == "MASS" else self.stiff_local(x)
            if which == "HELM":
                y += beta * self.mass_local(x)
            w = self.scatter(y)
            return w if mask is None else w * mask
        return apply

    def diagonal(self, which, beta=0.0, kappa=None):
        def squares(v, A, B):
            return self.tensor(v, [(A[c] * B[c]).T.contiguous() for c in range(3)])
        eye = torch.eye(self.p1, dtype=torch.float64, device="cuda") if self.colloc else self.J
        d = torch.zeros(self.E, self.p1, self.p1, self.p1, dtype=torch.float64, device="cuda")
        if which != "MASS":
            for a in range(3):
                for b in range(3):
                    v = self.g(a, b) if kappa is None else kappa * self.g(a, b)
                    d += squares(v, [self.D if c == a else eye for c in range(3)],
                                 [self.D if c == b else eye for c in range(3)])
        if which != "STIFF":
            d += (1.0 if which == "MASS" else beta) * squares(self.B, [eye] * 3, [eye] * 3)
        d = self.scatter(d)
        return d if self.free is None else d * self.free

    def pcg(self, apply, diag, b, iters, rtol=None):
        """Jacobi-PCG from zero: `iters` iterations, or fewer once every entry of
        b's rows has reached rtol."""
        inv = torch.where(diag != 0, 1.0 / diag, torch.zeros_like(diag))
        b = b if self.free is None else b * self.free
        x, r = torch.zeros_like(b), b.clone()
        z = inv * r
        p, rz, bb = z.clone(), r @ z, b @ b
        for k in range(iters):
            w = apply(p)
            alpha = rz / (p @ w)
            x += alpha * p
            r -= alpha * w
            z = inv * r
            new = r @ z
            p = z + (new / rz) * p
            rz = new
            if rtol is not None and k % 10 == 9 and float(r @ r) <= rtol * rtol * float(bb):
                break
        return x, float(torch.sqrt((r @ r) / bb))


def exact(case, seed):
    """What run() returns for these inputs, in plain FP64 torch."""
    s = _Plain(case, seed)
    v, kind, which, nc = s.vectors, case["kind"], _which(case), case["ncomp"]

    def rows(t):
        return t.double().reshape(nc, -1)

    def like(parts):
        return parts[0] if nc == 1 else torch.stack(parts)

    if kind in ("solve", "helmholtz", "mixed"):
        apply, diag = s.operator(which, case["beta"]), s.diagonal(which, case["beta"])
        iters, rtol = (case["iters"], None) if kind == "solve" else (8000, 3e-14)
        b = s.operator("MASS")(v["f"]) if kind == "mixed" else v["b"]
        got = [s.pcg(apply, diag, row, iters, rtol) for row in rows(b)]
        x = like([g[0] for g in got])
        return {"x": x, "rel_res": got[0][1], "iters": None} if kind == "solve" else {"x": x}
    if kind == "apply":
        apply = s.operator(which)
        return {"w": like([apply(u) for u in rows(v["u"])])}
    if kind == "local":
        f = s.mass_local if which == "MASS" else s.stiff_local
        shape = (s.E, s.p1, s.p1, s.p1)
        return {"w": torch.stack([f(u.reshape(shape)).reshape(s.E, -1) for u in rows(v["u"])])}
    kappa = v["kappa"].reshape(s.E, s.q, s.q, s.q)
    mass = s.operator("MASS", masked=False)
    d = [a - b for a, b in zip(rows(v["u"]), rows(v["target"]))]
    Md = [mass(x) for x in d]
    gk = torch.zeros_like(kappa)
    for lam, u in zip(rows(v["lam"]), rows(v["u"])):
        dl, du = s.gradient(s.gather(lam * s.free)), s.gradient(s.gather(u * s.free))
        for a in range(3):
            gk -= dl[a] * sum(s.g(a, b) * du[b] for b in range(3))
    return {"diag": s.diagonal("STIFF", kappa=kappa),
            "loss": 0.5 * float(sum(x @ y for x, y in zip(d, Md))),
            "grad": like(Md), "grad_kappa": gk.reshape(s.E, -1)}
