"""Cases whose speed is measured: calls of this framework as a solver's user makes them.

A case is a dict of plain values.  ``op`` names the entry point:

* ``apply``      one operator application (``Plan.apply``): the reduced operator that the Krylov
                 solves are made of, its transpose (the adjoint direction), the full rows (residuals)
* ``derivative`` one collocation derivative (``Plan.derivative``): fluxes in post-processing
* ``precond``    one application of the fast-diagonalisation preconditioner (``Plan.precond``)
* ``prolong``    a coarse solution onto the next level's grid (``prolong``)
* ``jacobian``   one Jacobian product of the nonlinear conductivity law (``Plan.newton_jacobian``)
* ``solve``      one preconditioned solve (``Plan.solve``)
* ``gradient``   a solve (zero face data) and the gradient of a loss with respect to log K
                 (``solve_logk``)
* ``homogenize`` apparent conductivities of several microstructures in one batch (``homogenize``)

Sizes are nodes per axis, ``edge`` the length of the box's edges.  The face sets: ``dirichlet`` (six Dirichlet faces), ``x`` (Dirichlet
x faces, zero flux elsewhere: the two-phase and homogenisation problems) and ``robin`` (Dirichlet
x faces, du/dn + u = g elsewhere: convective walls).
"""
import math

import numpy as np
import torch

from paper_2606_21410_amd import api

DEV = "cuda" if torch.cuda.is_available() else "cpu"
F64 = torch.float64
ALPHA = 0.5  # k(T) = K0 / (1 + ALPHA T) of the thermal problem
KC = 1.1     # mean conductivity given to the preconditioner
# with u prescribed on faces the right-hand side is dominated by the rows next to them: this leaves
# about 1e-10 in the solution
SOLVE_RTOL = 1e-13


def _case(op, n, **kw):
    c = {"op": op, "nx": n[0], "ny": n[1], "nz": n[2], "prec": "f64", "bc": "x", "edge": 1.0}
    c.update(kw)
    return c


def listed():
    return [
        # the smallest grid of the configurations: two launches, all latency
        _case("apply", (17, 17, 17), mode="reduced", name="apply f64 17"),
        # the metric grid of the benchmark
        _case("apply", (129, 129, 129), mode="reduced", name="apply f64 129"),
        # the largest level of the refinement chain
        _case("apply", (257, 257, 257), mode="reduced", name="apply f64 257"),
        # a box whose axes are resolved as the geometry asks, convective walls; the inner operator of
        # a mixed-precision solve runs in FP32
        _case("apply", (121, 81, 61), mode="reduced", prec="f32", bc="robin", name="apply f32 121x81x61"),
        # the adjoint direction on an even number of nodes
        _case("apply", (100, 100, 100), mode="transpose", name="transpose f64 100"),
        # residual with boundary rows, before and after a solve
        _case("apply", (65, 65, 65), mode="full", bc="robin", name="full f64 65"),
        # the preconditioner of one Krylov step at the metric grid
        _case("precond", (129, 129, 129), name="precond f64 129"),
        # the start of the next level of a refinement chain
        _case("prolong", (129, 129, 129), cx=65, cy=65, cz=65, name="prolong f64 65-129"),
        # one product inside Newton's LGMRES at the metric grid
        _case("jacobian", (129, 129, 129), name="jacobian f64 129"),
        # a mixed-precision solve
        _case("solve", (129, 129, 129), prec="mixed", name="solve mixed 129"),
        # the inverse problem's step: forward and adjoint solve
        _case("gradient", (33, 33, 33), name="gradient f64 33"),
        # microstructures of three sizes under three load cases each
        _case("homogenize", (49, 57, 65), prec="mixed", name="homogenize mixed 49-65"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _sizes(rng, lo, hi):
    """Half cubes of the usual transform sizes, a quarter cubes of any size, a quarter ragged boxes."""
    t = rng.random()
    if t < 0.5:
        n = rng.choice([m + 1 for m in (8, 16, 32, 48, 64, 96, 128, 192, 256) if lo <= m + 1 <= hi])
        return (n, n, n)
    if t < 0.75:
        n = _log_int(rng, lo, hi)
        return (n, n, n)
    return tuple(_log_int(rng, lo, hi) for _ in range(3))


def draw(rng):
    c = _draw(rng)
    if c["op"] != "homogenize":
        c["edge"] = round(rng.uniform(0.5, 2.0), 3)
    return c


def _draw(rng):
    op = rng.choices(["reduced", "transpose", "full", "derivative", "precond", "prolong", "jacobian", "solve",
                      "gradient", "homogenize"], [8, 2, 2, 1, 3, 2, 1, 3, 1, 1])[0]
    bc = rng.choice(["x", "dirichlet", "robin"])
    prec = rng.choice(["f64", "f64", "f32"])
    if op in ("reduced", "transpose", "full"):
        return _case("apply", _sizes(rng, 9, 257), mode=op, prec=prec, bc=bc)
    if op == "derivative":
        return _case("derivative", _sizes(rng, 9, 257), prec=prec, axis=rng.randrange(3))
    if op == "precond":
        return _case("precond", _sizes(rng, 9, 257), prec=prec, bc=bc)
    if op == "prolong":
        n = _sizes(rng, 17, 193)
        c = [max(9, int(round((m - 1) * rng.uniform(0.45, 0.8))) + 1) for m in n]
        return _case("prolong", n, cx=c[0], cy=c[1], cz=c[2])
    if op == "jacobian":
        return _case("jacobian", _sizes(rng, 9, 129), bc=bc)
    if op == "solve":
        return _case("solve", _sizes(rng, 17, 129), prec=rng.choice(["f64", "mixed"]))
    if op == "gradient":
        return _case("gradient", _sizes(rng, 17, 65))
    return _case("homogenize", tuple(_log_int(rng, 17, 49) for _ in range(3)), prec="mixed")


# --- inputs ---------------------------------------------------------------------------------

def _n(case):
    return case["nx"], case["ny"], case["nz"]


def _faces(bc):
    """(face types, Robin coefficients); 0 Dirichlet, 1 Neumann or Robin."""
    if bc == "dirichlet":
        return (0,) * 6, (0.0,) * 6
    if bc == "robin":
        return (0, 0, 1, 1, 1, 1), (0.0, 0.0, 1.0, 1.0, 1.0, 1.0)
    return (0, 0, 1, 1, 1, 1), (0.0,) * 6


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _smooth(n, gen, modes=12):
    """A smooth random field of unit variance on the collocation points of the unit box."""
    x = [0.5 - 0.5 * torch.cos(math.pi * torch.arange(m, device=DEV, dtype=F64) / (m - 1)) for m in n]
    k = 4.0 * torch.randn((modes, 3), generator=gen, device=DEV, dtype=F64)
    ph = 2 * math.pi * torch.rand((modes,), generator=gen, device=DEV, dtype=F64)
    out = torch.zeros(n, device=DEV, dtype=F64)
    for q in range(modes):
        out += torch.cos((k[q, 0] * x[0] + ph[q])[:, None, None] + (k[q, 1] * x[1])[None, :, None]
                         + (k[q, 2] * x[2])[None, None, :])
    return out * math.sqrt(2.0 / modes)


def _inputs(case, seed):
    """The call's input tensors, from the seed alone."""
    op, n, gen = case["op"], _n(case), _gen(seed)
    dt = torch.float32 if case["prec"] == "f32" else F64
    noise = lambda: torch.randn(n, generator=gen, device=DEV, dtype=F64).to(dt)
    if op == "homogenize":
        return {"K": [torch.exp(0.5 * _smooth((m, m, m), gen)) for m in n]}
    if op == "prolong":
        return {"uc": _smooth((case["cx"], case["cy"], case["cz"]), gen)}
    if op == "derivative":
        return {"u": noise()}
    if op == "precond":
        return {"r": noise()}
    s = {"K": torch.exp(0.5 * _smooth(n, gen)).to(dt)}
    if op == "apply":
        s["u"] = noise()
    elif op == "jacobian":
        s["T"] = 0.5 * torch.tanh(_smooth(n, gen))  # 1 + ALPHA T stays positive
        s["v"] = noise()
    else:
        s["f"] = _smooth(n, gen)
        if op == "gradient":
            s["w"] = _smooth(n, gen)
    return s


def _x_data(n, dt):
    """Packed face data: u = -1 / +1 on the x faces, zero flux elsewhere."""
    m = n[1] * n[2]
    g = torch.zeros(2 * (m + n[0] * n[2] + n[0] * n[1]), device=DEV, dtype=dt)
    g[:m] = -1.0
    g[m:2 * m] = 1.0
    return g


def prepare(case, seed):
    op, n = case["op"], _n(case)
    s = _inputs(case, seed)
    s["op"], s["case"] = op, case
    if op == "homogenize":
        grids = [((m, m, m), (0.0,) * 3, (1.0,) * 3, api.load_case((m, m, m), a, DEV)[0]) for m in n for a in range(3)]
        s["batch"] = api.Batch(grids, case["prec"], DEV)
        s["opts"] = api.SolveOptions(precond=True, rtol=SOLVE_RTOL)
        return s
    bc, robin = _faces(case["bc"])
    s["plan"] = api.Plan(n, hi=(case["edge"],) * 3, bc=bc, precision=case["prec"], device=DEV, robin=robin)
    if op == "apply":
        s["y"] = torch.empty_like(s["u"])
    elif op == "derivative":
        s["y"] = torch.empty_like(s["u"])
    elif op == "precond":
        s["out"] = torch.empty_like(s["r"])
    elif op == "prolong":
        s["coarse"] = api.Plan((case["cx"], case["cy"], case["cz"]), hi=(case["edge"],) * 3, bc=bc,
                               precision=case["prec"], device=DEV)
        s["uf"] = torch.empty(n, device=DEV, dtype=F64)
    elif op == "jacobian":
        s["y"] = torch.empty_like(s["v"])
    elif op == "solve":
        s["g"] = _x_data(n, F64)
        s["opts"] = api.SolveOptions(precond=True, rtol=SOLVE_RTOL)
    elif op == "gradient":
        s["g"] = torch.zeros(s["plan"].face_count(), device=DEV, dtype=F64)
        s["opts"] = api.SolveOptions(precond=True)
        s["logK"] = torch.log(s["K"]).requires_grad_(True)
    return s


def run(s):
    op = s["op"]
    if op == "apply":
        return s["plan"].apply(s["K"], s["u"], s["y"], s["case"]["mode"])
    if op == "derivative":
        return s["plan"].derivative(s["u"], s["case"]["axis"], s["y"])
    if op == "precond":
        return s["plan"].precond(s["r"], KC, s["out"])
    if op == "prolong":
        return api.prolong(s["coarse"], s["plan"], s["uc"], s["uf"])[0]
    if op == "jacobian":
        return s["plan"].newton_jacobian(s["K"], s["T"], s["v"], ALPHA, s["y"])
    if op == "solve":
        return s["plan"].solve(s["K"], s["f"], s["g"], opts=s["opts"])[0]
    if op == "gradient":
        u = api.solve_logk(s["plan"], s["logK"], s["f"], s["g"], s["opts"])
        s["logK"].grad = None
        u.backward(s["w"])
        return {"u": u.detach(), "grad": s["logK"].grad}
    tensors, _, us = api.homogenize(s["K"], precision=s["case"]["prec"], opts=s["opts"], batch=s["batch"])
    return {"K_app": np.array(tensors), "u": us}


def work(case):
    """Every input read and every output written once; the transforms' operations (two DCT-I of
    2.5 N log2 N each per derivative) where the number of derivatives is known."""
    op, n = case["op"], _n(case)
    pts = n[0] * n[1] * n[2]
    es = 4 if case["prec"] == "f32" else 8
    deriv = sum(5.0 * math.log2(m) + 3.0 for m in n)  # per point, one derivative along each axis
    if op == "apply":
        return {"bytes": 3 * es * pts, "flops": 2 * deriv * pts}
    if op == "derivative":
        return {"bytes": 2 * es * pts, "flops": (5.0 * math.log2(n[case["axis"]]) + 3.0) * pts}
    if op == "precond":
        # six dense contractions of the interior, halved by the even-odd symmetry
        return {"bytes": 2 * es * pts, "flops": 2.0 * sum(m - 2 for m in n) * pts}
    if op == "prolong":
        return {"bytes": es * (pts + case["cx"] * case["cy"] * case["cz"]), "flops": deriv * pts}
    if op == "jacobian":
        return {"bytes": 4 * es * pts, "flops": 3 * deriv * pts}
    if op == "solve":
        return {"bytes": 3 * 8 * pts, "flops": 2 * deriv * pts}
    if op == "gradient":
        return {"bytes": 5 * 8 * pts, "flops": 5 * deriv * pts}
    pts = sum(m ** 3 for m in n)
    return {"bytes": 8 * pts * 4, "flops": 3 * 2 * (15.0 * math.log2(max(n)) + 9.0) * pts}


# --- the same results in 64 bits, in plain torch ---------------------------------------------

def _diff(n, edge):
    """Collocation derivative at the ascending Chebyshev-Gauss-Lobatto points of [0, edge]."""
    N = n - 1
    i = np.arange(n)
    th = np.pi / (2 * N)
    dx = 2.0 * np.sin(th * (i[:, None] + i[None, :])) * np.sin(th * (i[:, None] - i[None, :]))
    c = np.where((i == 0) | (i == N), 2.0, 1.0) * (-1.0) ** i
    D = (c[:, None] / c[None, :]) / np.where(dx == 0.0, 1.0, dx)
    D[i, i] = 0.0
    D[i, i] = -D.sum(axis=1)
    return (2.0 / edge) * D


class _Axis:
    """D; L: interior values -> the pencil with its end values from the homogeneous face rows;
    M = D L; E: the interior rows of D; A = E M."""

    def __init__(self, n, edge, bc, sigma):
        D = _diff(n, edge)
        N = n - 1
        self.rows = np.zeros((2, n))  # the face rows, Dirichlet: the value itself
        rows = [(-D[0], sigma[0], 0), (D[N], sigma[1], N)]
        for q, (d, s, j) in enumerate(rows):
            if bc[q]:
                self.rows[q] = d
                self.rows[q, j] += s
            else:
                self.rows[q, j] = 1.0
        L = np.zeros((n, n - 2))
        L[1:N] = np.eye(n - 2)
        L[[0, N]] = -np.linalg.solve(self.rows[:, [0, N]], self.rows[:, 1:N])
        # end values from face data g = (lo, hi)
        self.H = np.zeros((n, 2))
        self.H[[0, N]] = np.linalg.inv(self.rows[:, [0, N]])
        self.bc = bc
        t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
        self.A = D[1:N] @ (D @ L)
        self.D, self.L, self.M, self.E, self.Ht, self.rowst = t(D), t(L), t(D @ L), t(D[1:N]), t(self.H), t(self.rows)


def _along(M, x, a):
    """M applied along axis a."""
    if a == 2:
        return (x.reshape(-1, x.shape[2]) @ M.t()).reshape(x.shape[0], x.shape[1], -1)
    if a == 0:
        return (M @ x.reshape(x.shape[0], -1)).reshape(-1, x.shape[1], x.shape[2])
    return torch.stack([M @ x[i] for i in range(x.shape[0])])


def _keep(x, a):
    """Every node along axis a, interior nodes along the other two."""
    s = [slice(1, -1)] * 3
    s[a] = slice(None)
    return x[tuple(s)]


def _axes(case, bc=None):
    f, r = _faces(case["bc"])
    f = bc or f
    return [_Axis(n, case["edge"], f[2 * a:2 * a + 2], r[2 * a:2 * a + 2]) for a, n in enumerate(_n(case))]


def _reduced(ax, K, x):
    return sum(_along(q.E, _keep(K, a) * _along(q.M, x, a), a) for a, q in enumerate(ax))


def _transposed(ax, K, w):
    return sum(_along(q.M.t(), _keep(K, a) * _along(q.E.t(), w, a), a) for a, q in enumerate(ax))


def _pad(x):
    return torch.nn.functional.pad(x, (1, 1, 1, 1, 1, 1))


class _Fdm:
    def __init__(self, ax):
        ev = [np.linalg.eig(q.A) for q in ax]
        assert all(np.abs(np.imag(l)).max() == 0.0 for l, _ in ev)
        t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
        self.V = [t(v.real) for _, v in ev]
        self.W = [t(np.linalg.inv(v.real)) for _, v in ev]
        l = [t(e.real) for e, _ in ev]
        self.lam = l[0][:, None, None] + l[1][None, :, None] + l[2][None, None, :]

    def __call__(self, r, kc=1.0, transpose=False):
        left, right = ([m.t() for m in self.V], [m.t() for m in self.W]) if transpose else (self.W, self.V)
        for a in range(3):
            r = _along(left[a], r, a)
        r = r / (kc * self.lam)
        for a in range(3):
            r = _along(right[a], r, a)
        return r


def _gmres(A, M, b, tol=2e-14, most=80, rounds=3):
    """Right-preconditioned GMRES, restarted from the true residual."""
    x = torch.zeros_like(b)
    nb = float(b.norm())
    for _ in range(rounds):
        r = b - A(x)
        beta = float(r.norm())
        if beta <= tol * nb:
            break
        V, Z = [r / beta], []
        H = np.zeros((most + 1, most))
        for j in range(most):
            Z.append(M(V[j]))
            w = A(Z[j])
            for _ in range(2):
                for i in range(j + 1):
                    h = float((V[i] * w).sum())
                    H[i, j] += h
                    w = w - h * V[i]
            H[j + 1, j] = float(w.norm())
            e = np.zeros(j + 2)
            e[0] = beta
            y, *_ = np.linalg.lstsq(H[:j + 2, :j + 1], e, rcond=None)
            if np.linalg.norm(H[:j + 2, :j + 1] @ y - e) <= 0.3 * tol * nb or j == most - 1:
                break
            V.append(w / H[j + 1, j])
        for j, c in enumerate(y):
            x = x + c * Z[j]
    return x


def _extend(ax, x, g):
    """Full nodal field from the interior values: end values along z, then y, then x; g[a]: the
    constant Dirichlet values of axis a, None for zero Neumann data."""
    for a in (2, 1, 0):
        q = ax[a]
        if g[a] is None:
            x = _along(q.L, x, a)
        else:
            shape = list(x.shape)
            shape[a] = 1
            x = torch.cat([torch.full(shape, g[a][0], device=DEV, dtype=F64), x,
                           torch.full(shape, g[a][1], device=DEV, dtype=F64)], dim=a)
    return x


def _rhs(ax, K, f, g):
    b = f[1:-1, 1:-1, 1:-1].clone()
    for a, q in enumerate(ax):
        if g[a] is not None:
            e = q.Ht @ torch.tensor(g[a], device=DEV, dtype=F64)
            s = (q.D @ e).reshape([-1 if d == a else 1 for d in range(3)])
            b = b - _along(q.E, _keep(K, a) * s, a)
    return b


def _solved(ax, K, f, g):
    P = _Fdm(ax)
    kc = float(K.mean())
    x = _gmres(lambda v: _reduced(ax, K, v), lambda r: P(r, kc), _rhs(ax, K, f, g))
    return _extend(ax, x, g), P, kc


def _full_rows(case, ax, K, u):
    y = _pad(sum(_along(q.E, _keep(K * _along(q.D, u, a), a), a) for a, q in enumerate(ax)))
    bc, _ = _faces(case["bc"])
    # a node on several faces carries the row of its first Dirichlet face, else of its first
    # Neumann face: written from the last in that order to the first
    order = [f for f in range(6) if not bc[f]] + [f for f in range(6) if bc[f]]
    for f in reversed(order):
        a, hi = f // 2, f % 2
        row = (ax[a].rowst[hi].reshape([-1 if d == a else 1 for d in range(3)]) * u).sum(dim=a)
        y.select(a, -1 if hi else 0).copy_(row)
    return y


def _cc_mean(F):
    """Clenshaw-Curtis average over the unit box."""
    for n in F.shape:
        N = n - 1
        k = np.arange(0, N + 1, 2)
        m = 2.0 / (1.0 - k.astype(float) ** 2)  # integrals of T_k over [-1, 1]
        j = np.arange(n)
        half = lambda i: np.where((i == 0) | (i == N), 0.5, 1.0)
        w = 2.0 / N * half(j) * (np.cos(np.pi * np.outer(j, k) / N) * (m * half(k))).sum(axis=1)
        F = (F * torch.from_numpy(0.5 * w).to(F.device).reshape([-1] + [1] * (F.dim() - 1))).sum(dim=0)
    return float(F)


def _bary(nc, nf):
    """Interpolation from nc to nf collocation points."""
    x, t = -np.cos(np.pi * np.arange(nc) / (nc - 1)), -np.cos(np.pi * np.arange(nf) / (nf - 1))
    w = (-1.0) ** np.arange(nc)
    w[[0, -1]] *= 0.5
    d = t[:, None] - x[None, :]
    hit = np.abs(d) < 1e-14
    q = w / np.where(hit, 1.0, d)
    q = np.where(hit.any(axis=1)[:, None], hit.astype(float), q)
    return torch.from_numpy(q / q.sum(axis=1, keepdims=True)).to(DEV)


def exact(case, seed):
    op = case["op"]
    s = {k: (v.double() if isinstance(v, torch.Tensor) else v) for k, v in _inputs(case, seed).items()}
    if op == "apply":
        ax = _axes(case)
        if case["mode"] == "full":
            return _full_rows(case, ax, s["K"], s["u"])
        f = _reduced if case["mode"] == "reduced" else _transposed
        return _pad(f(ax, s["K"], s["u"][1:-1, 1:-1, 1:-1].contiguous()))
    if op == "derivative":
        return _along(torch.from_numpy(_diff(_n(case)[case["axis"]], case["edge"])).to(DEV), s["u"], case["axis"])
    if op == "precond":
        return _pad(_Fdm(_axes(case))(s["r"][1:-1, 1:-1, 1:-1].contiguous(), KC))
    if op == "prolong":
        u = s["uc"]
        for a, (c, n) in enumerate(zip((case["cx"], case["cy"], case["cz"]), _n(case))):
            u = _along(_bary(c, n), u, a)
        return u
    if op == "jacobian":
        d = 1.0 + ALPHA * s["T"]
        k, k1 = s["K"] / d, -ALPHA * s["K"] / (d * d)
        v, y = s["v"][1:-1, 1:-1, 1:-1].contiguous(), 0.0
        for a, q in enumerate(_axes(case)):
            flux = _keep(k, a) * _along(q.M, v, a) + _keep(k1 * _along(q.D, s["T"], a), a) * _along(q.L, v, a)
            y = y + _along(q.E, flux, a)
        return _pad(y)
    if op == "homogenize":
        tensors, us = [], []
        for K in s["K"]:
            m = K.shape[0]
            cols = []
            for a in range(3):
                bc, _ = api.load_case((m, m, m), a, "cpu")
                ax = _axes({"nx": m, "ny": m, "nz": m, "edge": 1.0, "bc": "x"}, bc)
                g = [None] * 3
                g[a] = (0.0, 1.0)
                u, _, _ = _solved(ax, K, torch.zeros_like(K), g)
                us.append(u)
                cols.append([_cc_mean(K * _along(ax[b].D, u, b)) for b in range(3)])
            tensors.append(np.array(cols).T)
        return {"K_app": np.array(tensors), "u": us}
    ax = _axes(case)
    g = [(0.0, 0.0) if op == "gradient" else (-1.0, 1.0), None, None]
    K = s["K"]
    u, P, kc = _solved(ax, K, s["f"], g)
    if op == "solve":
        return u
    # transposed lift of the loss gradient, adjoint solve, sensitivity
    x = torch.zeros([m - 2 for m in K.shape], device=DEV, dtype=F64, requires_grad=True)
    _extend(ax, x, g).backward(s["w"])
    lam = _pad(_gmres(lambda v: _transposed(ax, K, v), lambda r: P(r, kc, True), x.grad))
    grad = -K * sum(_along(q.D, u, a) * _along(q.D.t(), lam, a) for a, q in enumerate(ax))
    return {"u": u, "grad": grad}
