"""The calls whose speed matters to a user of the spectral-element Poisson library.

A case names an entry point (`op`), a mesh, a polynomial degree and the
options of the context.  `prepare` sets the context up and makes the vectors,
`run` is one call as a solver program makes it, `exact` is the same result in
64 bits from the definitions of arXiv:2110.07663 (Sec. 2.1, Sec. 2.2, eqs. 1-9,
Algorithms 1 and 2) in plain torch, independent of the library.

Ranges: degrees 2..10 (the paper runs p = 7; the batched workload 5, 7, 9), 64
to 32768 elements, FP64 and FP32 vectors, FP16 geometric factors, FP16 Schwarz
operands, Jacobi, RAS and ASM smoothing, even and odd element counts.
"""
import math

import numpy as np
import torch

from paper_2110_07663_amd import sem
from paper_2110_07663_amd import workloads as wl

SCHEDULES = {2: (2, 1), 3: (3, 1), 4: (4, 2, 1), 5: (5, 3, 1), 6: (6, 3, 1), 7: (7, 3, 1),
             8: (8, 4, 1), 9: (9, 5, 1), 10: (10, 5, 1)}
MAX_NODES = 32 ** 3 * 8 ** 3  # E-vector entries of the largest mesh
SMOOTHERS = {"jacobi": sem.SMOOTH_JACOBI, "ras": sem.SMOOTH_RAS, "asm": sem.SMOOTH_ASM}
PRECISIONS = {"f64": sem.F64, "f32": sem.F32, "f16": sem.F16}


def listed():
    return [
        # the paper's operating point: pressure solve on 32^3 anisotropic
        # elements at p = 7, FP32 Chebyshev-RAS multigrid inside FP64 flexible CG
        {"name": "solve_32_p7_mixed", "op": "solve", "mesh": "layer", "nex": 32, "ney": 32,
         "nez": 32, "p": 7, "smoother": "ras", "prec": "f32", "krylov": "fcg", "coarse": "direct"},
        # an ordinary FP64 solve: 16^3 smoothly deformed elements, Chebyshev-Jacobi
        # multigrid, p = 1 level by Jacobi-PCG
        {"name": "solve_16_p7_f64_jacobi", "op": "solve", "mesh": "sin", "nex": 16, "ney": 16,
         "nez": 16, "p": 7, "smoother": "jacobi", "prec": "f64", "krylov": "pcg", "coarse": "pcg"},
        # the smallest solve (64 undeformed elements, p = 3): launches and latency
        {"name": "solve_4_p3_f64", "op": "solve", "mesh": "box", "nex": 4, "ney": 4, "nez": 4,
         "p": 3, "smoother": "jacobi", "prec": "f64", "krylov": "pcg", "coarse": "auto"},
        # several independent problems of uneven size and degree, four right sides
        # each, advanced together
        {"name": "batch_p579_mixed", "op": "batch", "problems": "8:5 8:7 12:7 8:9 12:5 12:9",
         "nrhs": 4, "smoother": "ras", "prec": "f32"},
        # one product with the outer FP64 operator at the paper's size
        {"name": "apply_A_32_p7_f64", "op": "apply_A", "mesh": "layer", "nex": 32, "ney": 32,
         "nez": 32, "p": 7, "prec": "f64"},
        # the smoother's FP32 operator at the batch's highest degree, odd element counts
        {"name": "apply_A_odd_p9_f32", "op": "apply_A", "mesh": "sin", "nex": 17, "ney": 13,
         "nez": 15, "p": 9, "prec": "f32"},
        # the Schwarz smoother's local solves at the paper's size, FP32
        {"name": "apply_S_32_p7_ras_f32", "op": "apply_S", "mesh": "layer", "nex": 32, "ney": 32,
         "nez": 32, "p": 7, "smoother": "ras", "prec": "f32"},
        # an all-FP64 smoothing step, the plain-precision solve's dominant phase
        {"name": "smooth_20_p7_ras_f64", "op": "smooth", "mesh": "layer", "nex": 20, "ney": 20,
         "nez": 20, "p": 7, "smoother": "ras", "prec": "f64", "order": 2},
        # additive Schwarz smoothing (the paper's Table 1 smoother), odd counts, FP32
        {"name": "smooth_odd_p7_asm_f32", "op": "smooth", "mesh": "sin", "nex": 11, "ney": 14,
         "nez": 13, "p": 7, "smoother": "asm", "prec": "f32", "order": 2},
        # a small smoothing step at a middle degree: launches count
        {"name": "smooth_8_p5_ras_f32", "op": "smooth", "mesh": "sin", "nex": 8, "ney": 8,
         "nez": 8, "p": 5, "smoother": "ras", "prec": "f32", "order": 2},
        # restriction of a residual and prolongation of a correction
        {"name": "transfer_20_p9_f32", "op": "transfer", "mesh": "layer", "nex": 20, "ney": 20,
         "nez": 20, "p": 9, "prec": "f32"},
        # one FP64 preconditioner application, p = 9 -> 5 -> 1
        {"name": "vcycle_odd_p9_ras_f64", "op": "vcycle", "mesh": "sin", "nex": 9, "ney": 7,
         "nez": 8, "p": 9, "smoother": "ras", "prec": "f64", "order": 2},
    ]


def _sides(rng, n_max, lo, hi):
    """Three element counts, log-uniform, with at most n_max elements."""
    while True:
        m = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        s = [max(2, round(m * rng.uniform(0.75, 1.3))) for _ in range(3)]
        if s[0] * s[1] * s[2] <= n_max:
            return s


def draw(rng):
    op = rng.choice(("apply_A", "apply_A", "apply_S", "apply_S", "smooth", "smooth", "transfer",
                     "vcycle", "solve", "batch"))
    if op == "batch":
        probs = " ".join("%d:%d" % (rng.choice((8, 12)), rng.choice((5, 7, 9)))
                         for _ in range(rng.randint(2, 5)))
        return {"op": op, "problems": probs, "nrhs": rng.randint(2, 4), "smoother": "ras",
                "prec": "f32"}
    p = rng.choice((2, 3, 4, 5, 6, 7, 7, 7, 8, 9, 9, 10))
    if op in ("vcycle", "solve"):
        p = rng.choice((3, 5, 7, 7, 9))
        s = _sides(rng, 3000, 4, 14)
    else:
        s = _sides(rng, MAX_NODES // (2 * (p + 1) ** 3), 4, 32)
    c = {"op": op, "mesh": "sin", "nex": s[0], "ney": s[1], "nez": s[2], "p": p,
         "prec": rng.choice(("f64", "f32", "f32"))}
    if rng.random() < 0.3:  # a cube, as the benchmark's meshes are
        c.update(mesh="layer", nex=min(s), ney=min(s), nez=min(s))
    if op == "apply_A" and c["prec"] == "f32" and rng.random() < 0.3:
        c["geom"] = "f16"
    if op in ("apply_S", "smooth", "vcycle", "solve"):
        c["smoother"] = rng.choice(("ras", "ras", "asm", "jacobi"))
    if op == "apply_S" and c["smoother"] == "ras" and c["prec"] == "f32" and rng.random() < 0.3:
        c["fdm"] = "f16"
    if op in ("smooth", "vcycle"):
        c["order"] = rng.choice((1, 2, 2, 3))
    if op == "vcycle":
        c["prec"] = "f64"
    if op == "solve":
        pcg = c["smoother"] == "jacobi" and c["prec"] == "f64"  # a symmetric preconditioner
        c.update(mesh="sin", krylov="pcg" if pcg else "fcg", coarse="auto")
    return c


# --- preparation and the calls -------------------------------------------------------------

def _mesh(case):
    """(xyz [E, (p_geom+1)^3, 3], p_geom) of the case's mesh."""
    n = (case["nex"], case["ney"], case["nez"])
    if case["mesh"] == "layer":
        return wl.layer_shift_vertices(n[0], seed=3), 1
    if case["mesh"] == "box":
        return wl.box_vertices(*n), 1
    pg = min(case["p"], 5)
    return wl.sampled_mesh(*n, _gll(pg)[0], wl.sin_map(0.05)), pg


# lambda~ of S A kept from an earlier run of the same problem (sem_opts.lambda_override);
# whole solves take theirs from the library's Arnoldi steps
def _lambda(case):
    if case.get("smoother", "jacobi") == "jacobi":
        return 2.6
    return 25.0 if case["mesh"] == "layer" else 2.2  # boxes fit sheared elements badly


def _options(case):
    op = case["op"]
    sched = SCHEDULES[case["p"]]
    whole = op in ("solve", "batch")
    o = sem.make_opts(
        schedule=sched, smoother=SMOOTHERS[case.get("smoother", "jacobi")],
        cheb_order=case.get("order", 2), smoother_prec=PRECISIONS[case["prec"]],
        fdm_prec=PRECISIONS[case.get("fdm", case["prec"])],
        krylov=sem.KRYLOV_PCG if case.get("krylov") == "pcg" else sem.KRYLOV_FCG,
        lambda_override=None if whole else [_lambda(case)] * 8,
        batch_rhs=case.get("nrhs", 0) if op == "batch" else 0,
        coarse_solver={"pcg": sem.COARSE_PCG, "direct": sem.COARSE_DIRECT}.get(
            case.get("coarse", "auto" if whole or op == "vcycle" else "pcg"), sem.COARSE_AUTO))
    if case.get("geom") == "f16":
        o.geom_prec = sem.F16
    return o


def _solver(case):
    xyz, pg = _mesh(case)
    return sem.Solver(case["nex"], case["ney"], case["nez"], xyz, pg, case["p"],
                      opts=_options(case))


def _problems(case):
    """The batch's problems as cases of their own."""
    out = []
    for word in case["problems"].split():
        n, p = (int(v) for v in word.split(":"))
        out.append(dict(case, mesh="sin", nex=n, ney=n, nez=n, p=p))
    return out


def _waves(seed, count=4):
    """Frequencies and amplitudes of a smooth field that vanishes on the unit cube's boundary."""
    rng = np.random.default_rng(seed)
    return [(rng.integers(1, 5, 3), float(rng.uniform(0.5, 1.0)) * (1 if rng.random() < 0.5 else -1))
            for _ in range(count)]


def _smooth_field(X, seed):
    u = torch.zeros_like(X[0])
    for (a, b, c), amp in _waves(seed):
        u += amp * torch.sin(math.pi * int(a) * X[0]) * torch.sin(math.pi * int(b) * X[1]) \
            * torch.sin(math.pi * int(c) * X[2])
    return u


def _random_global(case, p, seed):
    """U(-1, 1) on the level's node grid [nz, ny, nx], zero on the (Dirichlet) boundary."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    g = torch.Generator(device=dev).manual_seed(seed)
    shape = [case[k] * p + 1 for k in ("nez", "ney", "nex")]
    u = torch.rand(shape, generator=g, device=dev, dtype=torch.float64) * 2 - 1
    for d in range(3):
        u.select(d, 0).zero_()
        u.select(d, shape[d] - 1).zero_()
    return u


def _dtype(case):
    return torch.float64 if case["prec"] == "f64" else torch.float32


def prepare(case, seed):
    op = case["op"]
    if op == "batch":
        solvers = [_solver(c) for c in _problems(case)]
        bs = [[s.apply_A(_smooth_field(s.coords(), 1000 * seed + 10 * i + k))
               for k in range(case["nrhs"])] for i, s in enumerate(solvers)]
        return {"op": op, "s": solvers, "b": bs, "x": [[torch.zeros_like(b) for b in r] for r in bs]}
    s = _solver(case)
    st = {"op": op, "s": s}
    if op == "solve":
        st["b"] = s.apply_A(_smooth_field(s.coords(), seed))
        return st

    def vec(k, level=0, dtype=_dtype(case)):
        p = SCHEDULES[case["p"]][level]
        return s.gather(_random_global(case, p, 8 * seed + k), level).to(dtype)

    if op in ("apply_A", "apply_S"):
        st["u"] = vec(0)
        st["out"] = torch.empty_like(st["u"])
    elif op == "smooth":
        st["b"], st["x0"] = vec(0), vec(1)
        st["x"] = torch.empty_like(st["b"])
    elif op == "transfer":
        st["r"], st["x0"], st["e"] = vec(0), vec(1), vec(2, 1)
        st["x"], st["rc"] = torch.empty_like(st["r"]), torch.empty_like(st["e"])
    elif op == "vcycle":
        st["r"] = vec(0, dtype=torch.float64)
        st["z"] = torch.empty_like(st["r"])
    return st


def run(st):
    op, s = st["op"], st["s"]
    if op == "solve":
        return s.solve(st["b"], rtol=1e-8, maxit=300)[0]
    if op == "batch":
        for row in st["x"]:
            for x in row:
                x.zero_()
        sem.batch_solve(s, st["b"], st["x"], rtol=1e-8, maxit=200)
        return st["x"]
    if op == "apply_A":
        return s.apply_A(st["u"], out=st["out"])
    if op == "apply_S":
        return s.apply_S(st["u"], out=st["out"])
    if op == "smooth":
        return s.smooth(st["b"], st["x"].copy_(st["x0"]))
    if op == "transfer":  # both directions between the two finest levels
        return [s.restrict(st["r"], out=st["rc"]), s.prolong(st["e"], st["x"].copy_(st["x0"]))]
    return s.vcycle(st["r"], out=st["z"])


# --- what a pass cannot do without ------------------------------------------------------------

def _a_work(E, p, w, g):
    N = p + 1
    return np.array([E * N ** 3 * (2.0 * w + 6 * g), E * (12.0 * N ** 4 + 15 * N ** 3)])


def _s_work(E, p, w, smoother):
    N, pb = p + 1, p + 3
    if smoother == "jacobi":
        return np.array([E * N ** 3 * 3.0 * w, E * float(N ** 3)])
    return np.array([E * (2.0 * N ** 3 + 3 * pb * pb + 3 * pb) * w, E * (12.0 * pb ** 4 + pb ** 3)])


def _smooth_work(E, p, w, case, zero):
    k = case.get("order", 2)
    a, s = _a_work(E, p, w, w), _s_work(E, p, w, case["smoother"])
    return (k + (0 if zero else 1)) * a + (k + 1) * s


def _transfer_work(E, pf, pc, w):
    nf, nc = pf + 1, pc + 1
    flops = 2.0 * (nf * nc ** 3 + nf ** 2 * nc ** 2 + nf ** 3 * nc)
    return np.array([E * (nf ** 3 + nc ** 3) * float(w), E * flops])


def _vcycle_work(E, case, w):
    sched = SCHEDULES[case["p"]]
    total = np.zeros(2)
    for pf, pc in zip(sched, sched[1:]):
        total += _smooth_work(E, pf, w, case, True) + _smooth_work(E, pf, w, case, False)
        total += _a_work(E, pf, w, w) + 2 * _transfer_work(E, pf, pc, w)
    return total


def work(case):
    op = case["op"]
    if op == "batch":
        total = np.zeros(2)
        for c in _problems(case):
            total += case["nrhs"] * np.array(list(work(dict(c, op="solve", krylov="fcg")).values()))
        return {"bytes": float(total[0]), "flops": float(total[1])}
    E, p = case["nex"] * case["ney"] * case["nez"], case["p"]
    w = 8 if case["prec"] == "f64" else 4
    if op == "apply_A":
        t = _a_work(E, p, w, 2 if case.get("geom") == "f16" else w)
    elif op == "apply_S":
        t = _s_work(E, p, w, case["smoother"])
    elif op == "smooth":
        t = _smooth_work(E, p, w, case, False)
    elif op == "transfer":
        t = 2 * _transfer_work(E, p, SCHEDULES[p][1], w)
        t[0] += E * (p + 1) ** 3 * w
    elif op == "vcycle":
        t = _vcycle_work(E, case, w)
    else:  # outer iterations to 1e-8: about 50 on the strongly sheared mesh, 10 on the smooth ones
        its = 50 if case["mesh"] == "layer" else 10
        t = its * (_vcycle_work(E, case, w) + _a_work(E, p, 8, 8) + [E * (p + 1) ** 3 * 72.0, 0])
    return {"bytes": float(t[0]), "flops": float(t[1])}


# --- the same results in 64 bits, from the definitions ----------------------------------------

def _gll(p):
    """GLL nodes and weights of degree p: roots of (1 - x^2) P_p'."""
    c = np.zeros(p + 1)
    c[p] = 1
    P = np.polynomial.legendre.Legendre(c)
    x = np.sort(np.concatenate([[-1.0], P.deriv().roots().real, [1.0]])) if p > 1 else np.array([-1.0, 1.0])
    for _ in range(3):  # polish the interior roots
        x[1:-1] -= P.deriv()(x[1:-1]) / P.deriv(2)(x[1:-1]) if p > 1 else 0
    return x, 2.0 / (p * (p + 1) * P(x) ** 2)


def _cardinal(x, y):
    """J[i, j]: cardinal polynomial j on the nodes x, at y_i."""
    return np.array([[np.prod([(b - x[m]) / (x[j] - x[m]) for m in range(len(x)) if m != j])
                      for j in range(len(x))] for b in y])


def _derivative(x):
    n = len(x)
    c = [np.prod([x[j] - x[m] for m in range(n) if m != j]) for j in range(n)]
    D = np.array([[0.0 if i == j else c[i] / (c[j] * (x[i] - x[j])) for j in range(n)] for i in range(n)])
    return D - np.diag(D.sum(1))


def _along(M, u, d):
    """u[e, k, j, i] times the matrix M along direction d (0: i, 1: j, 2: k)."""
    return torch.movedim(torch.movedim(u, 3 - d, 3) @ M.T, 3, 3 - d)


class _Level:
    """One level of the hierarchy in FP64: geometry, operator, smoother."""

    def __init__(self, case, p):
        self.dev = "cuda" if torch.cuda.is_available() else "cpu"
        self.n = n = (case["nex"], case["ney"], case["nez"])
        self.p, self.E, self.case = p, n[0] * n[1] * n[2], case
        xyz, pg = _mesh(case)
        x, w = _gll(p)
        self.x, self.D = x, self.t(_derivative(x))
        self.w = w
        J = self.t(_cardinal(_gll(pg)[0], x))
        X = self.t(xyz).permute(2, 0, 1).reshape(3, self.E, pg + 1, pg + 1, pg + 1)
        self.X = torch.stack([self.cube(J, X[a]) for a in range(3)])
        e = torch.arange(self.E, device=self.dev)
        self.pos = (e % n[0], (e // n[0]) % n[1], e // (n[0] * n[1]))
        self.gid, ok = self.grid(torch.arange(p + 1, device=self.dev))
        self.shape = tuple(n[d] * p + 1 for d in (2, 1, 0))
        self.mult = self.gather(self.scatter(torch.ones(self.gid.shape, device=self.dev, dtype=torch.float64)))
        m = torch.zeros(self.shape, device=self.dev, dtype=torch.float64)
        m[1:-1, 1:-1, 1:-1] = 1
        self.mask = self.gather(m.reshape(-1))

    def t(self, a):
        return torch.as_tensor(a, dtype=torch.float64, device=self.dev)

    def cube(self, J, u):
        for d in range(3):
            u = _along(J, u, d)
        return u

    def grid(self, r):
        """Global indices of the local offsets r (per direction) of every element, and which exist."""
        g = [self.pos[d][:, None] * self.p + r for d in range(3)]
        n = [self.n[d] * self.p + 1 for d in range(3)]
        ok = [(g[d] >= 0) & (g[d] < n[d]) for d in range(3)]
        ok = ok[2][:, :, None, None] & ok[1][:, None, :, None] & ok[0][:, None, None, :]
        gid = (g[2][:, :, None, None] * n[1] + g[1][:, None, :, None]) * n[0] + g[0][:, None, None, :]
        return torch.where(ok, gid, 0), ok

    def scatter(self, u):
        out = torch.zeros(math.prod(self.shape), device=self.dev, dtype=torch.float64)
        return out.index_add_(0, self.gid.reshape(-1), u.reshape(-1))

    def gather(self, g):
        return g[self.gid]

    def assemble(self, u):
        return self.mask * self.gather(self.scatter(u))

    def factors(self):
        """(rr, rs, rt, ss, st, tt) of w det(J) J^-1 J^-T at every point (Sec. 2.1)."""
        c = [[_along(self.D, self.X[a], b) for b in range(3)] for a in range(3)]  # dx_a/dr_b
        cof = [[c[(a + 1) % 3][(b + 1) % 3] * c[(a + 2) % 3][(b + 2) % 3]
                - c[(a + 1) % 3][(b + 2) % 3] * c[(a + 2) % 3][(b + 1) % 3] for b in range(3)] for a in range(3)]
        det = sum(c[0][b] * cof[0][b] for b in range(3))
        w = self.t(self.w)
        sc = w[:, None, None] * w[:, None] * w / det  # dr_b/dx_a = cof[a][b] / det
        return [sc * sum(cof[a][i] * cof[a][j] for a in range(3))
                for i, j in ((0, 0), (0, 1), (0, 2), (1, 1), (1, 2), (2, 2))]

    def local_A(self, u):
        if not hasattr(self, "G"):
            self.G = self.factors()
        g = self.G
        r, s, t = (_along(self.D, u, d) for d in range(3))
        Dt = self.D.T
        return _along(Dt, g[0] * r + g[1] * s + g[2] * t, 0) + _along(Dt, g[1] * r + g[3] * s + g[4] * t, 1) \
            + _along(Dt, g[2] * r + g[4] * s + g[5] * t, 2)

    def A(self, u):
        return self.assemble(self.local_A(u))

    def diagonal(self):
        if not hasattr(self, "G"):
            self.G = self.factors()
        g, D2, d = self.G, (self.D ** 2).T, torch.diagonal(self.D)
        out = _along(D2, g[0], 0) + _along(D2, g[3], 1) + _along(D2, g[5], 2)
        out = out + 2 * (g[1] * d * d[:, None] + g[2] * d * d[:, None, None] + g[4] * d[:, None] * d[:, None, None])
        return self.gather(self.scatter(out))

    def schwarz(self):
        """S and lambda of the extended 1D problems of every element (eqs. 5-7)."""
        p, n = self.p, self.n
        pb = p + 3
        c = self.X[:, :, ::p][:, :, :, ::p][..., ::p].cpu().numpy()
        K1 = (self.D.T @ torch.diag(self.t(self.w)) @ self.D).cpu().numpy()
        S, lam = [], []
        for d in range(3):
            ax = 4 - d  # the direction's axis in [3, E, 2, 2, 2]
            edge = np.sqrt((np.diff(c, axis=ax) ** 2).sum(0)).reshape(self.E, 4).mean(1)
            pos = self.pos[d].cpu().numpy()
            step = (1, n[0], n[0] * n[1])[d]
            has = [pos > 0, np.ones(self.E, bool), pos < n[d] - 1]
            idx = np.arange(self.E)
            K, M = np.zeros((self.E, pb, pb)), np.zeros((self.E, pb))
            for t in range(3):
                L = edge[np.clip(idx + (t - 1) * step, 0, self.E - 1)]
                q = np.arange(pb)
                a = p - 1 + q - t * p
                q, a = q[(a >= 0) & (a <= p)], a[(a >= 0) & (a <= p)]
                K[:, q[:, None], q] += np.where(has[t], 2 / L, 0)[:, None, None] * K1[np.ix_(a, a)]
                M[:, q] += np.where(has[t], L / 2, 0)[:, None] * self.w[a]
            cut = np.zeros((self.E, pb), bool)  # no neighbour, and the Dirichlet face node
            cut[:, 0] = cut[:, 1] = ~has[0]
            cut[:, -1] = cut[:, -2] = ~has[2]
            mh = np.where(cut, 0, 1 / np.sqrt(np.where(cut, 1, M)))
            C = mh[:, :, None] * K * mh[:, None, :]
            top = 10 * np.abs(C).sum((1, 2))  # decoupled nodes: eigenvalues above all others
            C[:, np.arange(pb), np.arange(pb)] += np.where(cut, top[:, None], 0)
            l, V = np.linalg.eigh(C)
            S.append(self.t(mh[:, :, None] * V))
            lam.append(self.t(np.where(l > 0.9 * top[:, None], np.inf, l)))
        return S, lam

    def S(self, r):
        """The smoother on a consistent vector (eqs. 4, 8, 9)."""
        kind = self.case["smoother"]
        if kind == "jacobi":
            if not hasattr(self, "diag"):
                self.diag = self.diagonal()
            return self.mask * r / self.diag
        if not hasattr(self, "fdm"):
            self.fdm = self.schwarz()
            self.box, self.ok = self.grid(torch.arange(-1, self.p + 2, device=self.dev))
        S, lam = self.fdm
        g = torch.zeros(math.prod(self.shape), device=self.dev, dtype=torch.float64)
        g[self.gid.reshape(-1)] = r.reshape(-1)
        u = torch.where(self.ok, g[self.box], 0.0)
        one = lambda M, v, d: torch.movedim(  # noqa: E731
            torch.matmul(torch.movedim(v, 3 - d, 3).reshape(self.E, -1, self.p + 3), M).reshape(
                (self.E,) + (self.p + 3,) * 3), 3, 3 - d)
        for d in range(3):
            u = one(S[d], u, d)
        u = u / (lam[2][:, :, None, None] + lam[1][:, None, :, None] + lam[0][:, None, None, :])
        for d in range(3):
            u = one(S[d].transpose(1, 2).contiguous(), u, d)
        if kind == "ras":
            return self.assemble(u[:, 1:-1, 1:-1, 1:-1] / self.mult)
        z = torch.zeros_like(g)
        z.index_add_(0, self.box.reshape(-1), torch.where(self.ok, u, 0.0).reshape(-1))
        cnt = torch.zeros_like(g).index_add_(0, self.box.reshape(-1), self.ok.double().reshape(-1))
        return self.mask * self.gather(z / cnt)

    def smooth(self, b, x):
        """x + the Chebyshev correction of Algorithm 2 (x None: zero)."""
        lt = _lambda(self.case)
        theta, delta = 0.5 * (1.1 + 0.1) * lt, 0.5 * (1.1 - 0.1) * lt
        sigma = theta / delta
        rho = 1 / sigma
        r = self.S(b if x is None else b - self.A(x))
        d = r / theta
        e = torch.zeros_like(b)
        for _ in range(self.case.get("order", 2)):
            e = e + d
            r = r - self.S(self.A(d))
            new = 1 / (2 * sigma - rho)
            d = new * rho * d + (2 * new / delta) * r
            rho = new
        return e + d if x is None else x + e + d

    def to_coarse(self, C, r):
        return C.assemble(self.cube(self.t(_cardinal(C.x, self.x)).T, r / self.mult))

    def from_coarse(self, C, e):
        return self.cube(self.t(_cardinal(C.x, self.x)), e)

    def solve_coarse(self, b):
        """The lowest level's system, assembled dense."""
        m = (self.p + 1) ** 3
        n = math.prod(self.shape)
        cols = torch.stack([self.local_A(torch.eye(m, device=self.dev, dtype=torch.float64)[c].reshape(
            1, *self.gid.shape[1:]).expand(self.E, -1, -1, -1)).reshape(self.E, m) for c in range(m)], 2)
        gid = self.gid.reshape(self.E, m)
        A = torch.zeros(n * n, device=self.dev, dtype=torch.float64)
        A.index_add_(0, (gid[:, :, None] * n + gid[:, None, :]).reshape(-1), cols.reshape(-1))
        free = torch.zeros(n, device=self.dev, dtype=torch.bool)
        free[gid.reshape(-1)] = self.mask.reshape(-1) > 0
        rhs = torch.zeros(n, device=self.dev, dtype=torch.float64)
        rhs[gid.reshape(-1)] = b.reshape(-1)
        x = torch.zeros_like(rhs)
        x[free] = torch.linalg.solve(A.reshape(n, n)[free][:, free], rhs[free])
        return self.gather(x)


def _vcycle(levels, b):
    L = levels[0]
    if len(levels) == 1:
        return L.solve_coarse(b)
    x = L.smooth(b, None)
    e = _vcycle(levels[1:], L.to_coarse(levels[1], b - L.A(x)))
    return L.smooth(b, x + L.from_coarse(levels[1], e))


def exact(case, seed):
    op, sched = case["op"], SCHEDULES.get(case.get("p"))
    if op == "batch":  # the right sides are A u of known fields u
        return [[_smooth_field(L.X.reshape(3, -1), 1000 * seed + 10 * i + k) for k in range(case["nrhs"])]
                for i, L in enumerate(_Level(c, c["p"]) for c in _problems(case))]
    L = _Level(case, case["p"])
    if op == "solve":
        return _smooth_field(L.X.reshape(3, -1), seed)

    def vec(k, level=L, dtype=_dtype(case)):
        return level.gather(_random_global(case, level.p, 8 * seed + k).reshape(-1)).to(dtype).double()

    if op == "apply_A":
        return L.A(vec(0)).reshape(-1)
    if op == "apply_S":
        return L.S(vec(0)).reshape(-1)
    if op == "smooth":
        return L.smooth(vec(0), vec(1)).reshape(-1)
    if op == "transfer":
        C = _Level(case, sched[1])
        return [L.to_coarse(C, vec(0)).reshape(-1), (vec(1) + L.from_coarse(C, vec(2, C))).reshape(-1)]
    if math.prod(case[k] + 1 for k in ("nex", "ney", "nez")) > 4000:
        return None  # the dense coarse system would be too large
    levels = [L] + [_Level(case, p) for p in sched[1:]]
    return _vcycle(levels, vec(0, dtype=torch.float64)).reshape(-1)
