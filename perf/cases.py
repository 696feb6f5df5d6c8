"""The work that users of this package have it do, as cases to be timed.

A user solves QPs (whole `solve` calls on a problem that stays on the device, and one-shot solves
that set a small problem up first), solves linear systems with the reduced KKT matrix (`pcg`), and
trains or evaluates the learned preconditioner (`hutchinson` targets, `loss_grad`, and a first
`forward` on a new instance, setup included). The sizes are the package's benchmark, parity and
training sizes, from a few hundred variables, where latency counts, to 10^8 matrix entries; both
arithmetics and both preconditioners occur. Problems are drawn on the GPU (the distributions of
`paper_1912_04263_amd.problems`), so that the largest instance is made in seconds.

Mixed-precision iterates are held in float32 on the device, so their results are returned as such.
"""
import math

import numpy as np
import torch

from paper_1912_04263_amd import problems, qpg
from paper_1912_04263_amd.problems import sp

INF = float("inf")
F64 = torch.float64


# ------------------------------------------------------------------------------------- the cases

def listed():
    return [
        # model predictive control: one small step, solved again and again; latency is all
        dict(name="solve_control_n320_fp64", kind="solve", family="control", a=20, b=10, t=10, dens=0.3, mixed=False),
        # the plain random QP of the benchmark: a small dense-ish problem
        dict(name="solve_random_n200_fp64", kind="solve", family="random", a=200, b=400, dens=0.15, mixed=False),
        # a program that solves one small problem once: setup and solve together
        dict(name="oneshot_svm_4000x100_fp64", kind="oneshot", family="svm", a=4000, b=100, dens=0.1, mixed=False),
        # a small regression in mixed precision
        dict(name="solve_lasso_2000x200_mixed", kind="solve", family="lasso", a=2000, b=200, dens=0.05, mixed=True),
        # the benchmark's Lasso: 10^7 entries, one PCG step per ADMM step
        dict(name="solve_lasso_100kx10k_fp64", kind="solve", family="lasso", a=100_000, b=10_000, dens=0.01,
             mixed=False),
        # the random class at the middle of its range, rows scattered over all columns
        dict(name="solve_random_n20000_mixed", kind="solve", family="random", a=20_000, b=200_000, dens=1e-3,
             mixed=True),
        # the benchmark's headline: 10^8 entries, bound by memory
        dict(name="solve_svm_1Mx10k_mixed", kind="solve", family="svm", a=1_000_000, b=10_000, dens=0.01, mixed=True),
        # linear systems with the learned diagonal, as the training driver's evaluation solves them
        dict(name="pcg_portfolio_20kx200_learned", kind="pcg", family="portfolio", a=20_000, b=200, dens=0.5,
             mixed=False, learned=True, eps=1e-10, rho=0.1),
        # the benchmark's portfolio matrix: many PCG steps over 5*10^7 entries
        dict(name="pcg_portfolio_100kx1k_fp64", kind="pcg", family="portfolio", a=100_000, b=1_000, dens=0.5,
             mixed=False, learned=False, eps=1e-8, rho=0.1),
        # training targets of one instance
        dict(name="hutchinson_portfolio_20kx200", kind="hutchinson", family="portfolio", a=20_000, b=200, dens=0.5,
             probes=16, eps=1e-8, rho=0.1),
        # one training step: forward and backward through the message-passing network
        dict(name="train_portfolio_20kx200", kind="train", family="portfolio", a=20_000, b=200, dens=0.5, rho=0.1),
        # a new instance in the training loop: setup, graph and the first forward pass
        dict(name="instance_svm_20kx1k", kind="instance", family="svm", a=20_000, b=1_000, dens=0.1, rho=1.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))))) | 1 if rng.random() < 0.5 else \
        int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve"] * 5 + ["oneshot", "pcg", "pcg", "hutchinson", "train", "instance"])
    mixed = rng.random() < 0.5
    rho = round(10.0 ** rng.uniform(-2, 1), 4)
    if kind == "solve":
        family = rng.choice(["control", "random", "random", "lasso", "lasso", "svm", "svm", "equality"])
        if family == "control":
            return dict(kind=kind, family=family, a=_log_int(rng, 6, 60), b=_log_int(rng, 3, 30), t=_log_int(rng, 5, 20),
                        dens=0.3, mixed=False)
        if family == "equality":
            a = _log_int(rng, 200, 50_000)
            return dict(kind=kind, family=family, a=a, b=a // 2, dens=min(0.15, 40.0 / a), mixed=False)
        if family == "random":
            a = _log_int(rng, 50, 50_000)
            b = int(a * rng.uniform(2, 10))
            return dict(kind=kind, family=family, a=a, b=b, dens=min(0.15, 20.0 / a), mixed=mixed)
        if family == "lasso":
            b = _log_int(rng, 50, 8_000)
            return dict(kind=kind, family=family, a=10 * b + rng.randrange(10), b=b, dens=min(0.15, 100.0 / b),
                        mixed=mixed)
        b = _log_int(rng, 50, 5_000)
        return dict(kind=kind, family=family, a=int(b * rng.uniform(20, 80)), b=b, dens=min(0.15, 100.0 / b),
                    mixed=mixed)
    if kind == "oneshot":
        family = rng.choice(["random", "svm", "lasso"])
        b = _log_int(rng, 40, 1_000)
        a = b if family == "random" else int(b * rng.uniform(10, 40))
        return dict(kind=kind, family=family, a=a, b=3 * a if family == "random" else b, dens=min(0.15, 30.0 / b),
                    mixed=False)
    if kind == "pcg":
        family = rng.choice(["portfolio", "portfolio", "random", "lasso"])
        if family == "portfolio":
            b = _log_int(rng, 20, 600)
            return dict(kind=kind, family=family, a=100 * b + rng.randrange(100), b=b, dens=0.5, mixed=False,
                        learned=rng.random() < 0.5, eps=1e-10, rho=rho)
        b = _log_int(rng, 100, 5_000)
        return dict(kind=kind, family=family, a=b if family == "random" else 10 * b, b=5 * b if family == "random" else b,
                    dens=min(0.15, 20.0 / b), mixed=False, learned=False, eps=1e-10, rho=rho)
    if kind == "hutchinson":
        b = _log_int(rng, 20, 300)
        return dict(kind=kind, family="portfolio", a=100 * b + rng.randrange(100), b=b, dens=0.5,
                    probes=rng.randrange(3, 33), eps=1e-8, rho=rho)
    family = rng.choice(["portfolio", "svm", "lasso"])
    b = _log_int(rng, 40, 400)
    return dict(kind=kind, family=family, a=(100 if family == "portfolio" else 20) * b + rng.randrange(50), b=b,
                dens=0.5 if family == "portfolio" else min(0.2, 100.0 / b), rho=rho)


# ------------------------------------------------------------------------------ problems (inputs)

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _pattern(g, rows, cols, dens):
    """Rows and columns of about dens*rows*cols distinct uniform positions, sorted by column."""
    if dens >= 0.2:
        pos = torch.nonzero(torch.rand(rows * cols, generator=g, device="cuda") < dens).reshape(-1)
        return pos % rows, pos // rows
    count = max(1, int(round(rows * cols * dens)))
    pos = torch.randint(0, rows * cols, (count,), generator=g, device="cuda")
    pos = torch.unique(pos)
    return pos % rows, pos // rows


def _randn(g, n):
    return torch.randn(n, generator=g, device="cuda", dtype=F64)


def _rand(g, n):
    return torch.rand(n, generator=g, device="cuda", dtype=F64)


def _csc(rows, cols, parts):
    """SciPy CSC matrix from (row, column, value) parts on the GPU (no position twice)."""
    r, c, v = (torch.cat([p[k] for p in parts]) for k in range(3))
    order = torch.argsort(c * rows + r)
    indptr = np.zeros(cols + 1, np.int32)
    indptr[1:] = torch.cumsum(torch.bincount(c, minlength=cols), 0).cpu().numpy()
    return sp.csc_matrix((v[order].cpu().numpy(), r[order].to(torch.int32).cpu().numpy(), indptr), shape=(rows, cols))


def _eye(n, r0, c0, value=1.0):
    i = torch.arange(n, device="cuda")
    return i + r0, i + c0, torch.full((n,), float(value), device="cuda", dtype=F64)


def _host(*vs):
    return [v.cpu().numpy() for v in vs]


def _gram(g, n, dens):
    """Upper triangle of M M^T + 0.01 I, M an n x n Bernoulli matrix with N(0, 1) entries."""
    r, c = _pattern(g, n, n, dens)
    M = _csc(n, n, [(r, c, _randn(g, r.numel()))]).tocsr()
    P = sp.triu(M @ M.T + 0.01 * sp.identity(n, format="csr"), format="csc")
    P.sort_indices()
    return P


def _problem(case, seed):
    """(P_triu, q, A, l, u) of the case's family, in the solver's input form."""
    f, a, b, dens = case["family"], case["a"], case["b"], case["dens"]
    if f == "control":  # a states, b inputs, horizon t
        p = problems.control_qp(a, b, case["t"], dens, seed)
        return p.P_triu, p.q, p.A, p.l, p.u
    g = _gen(seed)
    if f in ("random", "equality"):  # a variables, b rows
        P = _gram(g, a, min(dens, 4.47 / a) if dens < 0.15 else dens)
        r, c = _pattern(g, b, a, dens)
        v = _randn(g, r.numel())
        A = _csc(b, a, [(r, c, v)])
        q, x0 = _host(_randn(g, a), _randn(g, a))
        if f == "equality":
            rhs = A @ x0
            return P, q, A, rhs, rhs.copy()
        lo, up = _host(-_rand(g, b), _rand(g, b))
        return P, q, A, lo, up
    if f == "portfolio":  # a assets, b factors
        r, c = _pattern(g, b, a, dens)  # the factor matrix transposed
        A = _csc(b + 1 + a, a + b, [(r, c, _randn(g, r.numel())), _eye(b, 0, a, -1.0),
                                    (torch.full((a,), b, device="cuda"), torch.arange(a, device="cuda"),
                                     torch.ones(a, device="cuda", dtype=F64)), _eye(a, b + 1, 0)])
        d, mu = _host(2.0 * math.sqrt(b) * _rand(g, a), _randn(g, a))
        P = sp.diags(np.concatenate([d, np.full(b, 2.0)]), format="csc")
        q = np.concatenate([-mu, np.zeros(b)])
        lo = np.concatenate([np.zeros(b), [1.0], np.zeros(a)])
        up = np.concatenate([np.zeros(b), [1.0], np.full(a, INF)])
        return P, q, A, lo, up
    r, c = _pattern(g, a, b, dens)  # a data rows, b features
    if f == "svm":
        label = torch.where(torch.arange(a, device="cuda") < a // 2, 1.0, -1.0).to(F64)
        v = label[r] * (_randn(g, r.numel()) / math.sqrt(b) + label[r] / b)
        A = _csc(2 * a, b + a, [(r, c, v), _eye(a, 0, b, -1.0), _eye(a, a, b)])
        P = sp.csc_matrix((np.full(b, 2.0), np.arange(b, dtype=np.int32),
                           np.minimum(np.arange(a + b + 1), b).astype(np.int32)), shape=(a + b, a + b))
        q = np.concatenate([np.zeros(b), np.ones(a)])
        lo = np.concatenate([np.full(a, -INF), np.zeros(a)])
        up = np.concatenate([np.full(a, -1.0), np.full(a, INF)])
        return P, q, A, lo, up
    assert f == "lasso"
    v = _randn(g, r.numel())
    x, noise = _host(_randn(g, b) / math.sqrt(b), _randn(g, a))
    x[np.random.default_rng(seed).permutation(b)[: b // 2]] = 0.0
    rhs = _csc(a, b, [(r, c, v)]) @ x + noise
    A = _csc(a + 2 * b, a + 2 * b, [(r, c, v), _eye(a, 0, b, -1.0), _eye(b, a, 0), _eye(b, a, a + b, -1.0),
                                    _eye(b, a + b, 0), _eye(b, a + b, a + b)])
    lam = float(np.max(np.abs(A[:a, :b].T @ rhs))) / 5.0
    d = np.zeros(a + 2 * b)
    d[b:a + b] = 2.0
    P = sp.diags(d, format="csc")
    P.eliminate_zeros()
    q = np.concatenate([np.zeros(a + b), np.full(b, lam)])
    lo = np.concatenate([rhs, np.full(b, -INF), np.zeros(b)])
    up = np.concatenate([rhs, np.zeros(b), np.full(b, INF)])
    return P, q, A, lo, up


def _settings(case):
    kw = dict(precision="mixed" if case.get("mixed") else "fp64")
    if case.get("learned"):
        kw.update(precond="learned", precond_weights=qpg.load_weights("portfolio_h32"))
    return kw


# ---------------------------------------------------------------------------------- state and run

def prepare(case, seed):
    prob = _problem(case, seed)
    kind = case["kind"]
    rng = np.random.default_rng(seed)
    st = dict(case=case, prob=prob if kind in ("oneshot", "instance") else None)
    if kind not in ("oneshot", "instance"):
        st["solver"] = qpg.Solver(*prob, stream=torch.cuda.current_stream().cuda_stream, **_settings(case))
    n = prob[2].shape[1]
    if kind == "pcg":
        st["solver"].set_rho(case["rho"])
        st["b"] = rng.standard_normal(n)
    if kind == "hutchinson":
        st["signs"] = rng.choice(np.array([-1, 1], dtype=np.int8), size=(case["probes"], n))
    if kind in ("train", "instance"):
        st["net"] = qpg.Net(_weights(case), bf16=True)
        st["target"] = np.abs(rng.normal(0.0, 0.5, n)).astype(np.float32)
    return st


def _weights(case):
    return qpg.load_weights("portfolio_h32" if case["family"] == "portfolio" else case["family"] + "_h32")


def _iterates(solver, mixed):
    x, y = torch.from_numpy(solver.x()), torch.from_numpy(solver.y())
    return (x.float(), y.float()) if mixed else (x, y)


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "solve":
        info = st["solver"].solve()
        x, y = _iterates(st["solver"], case["mixed"])
        return dict(x=x, y=y, iters=info.iter)
    if kind == "oneshot":
        x, y, info = qpg.solve(*st["prob"], **_settings(case))
        return dict(x=x, y=y, iters=info.iter)
    if kind == "pcg":
        x, it, _, _ = st["solver"].pcg(st["b"], eps=case["eps"], max_iter=5000)
        return dict(x=x, iters=it)
    if kind == "hutchinson":
        return dict(diag=st["solver"].hutchinson(st["signs"], case["rho"], eps=case["eps"], max_iter=2000))
    if kind == "train":
        loss, grad = st["net"].loss_grad(st["solver"], case["rho"], st["target"])
        return dict(loss=torch.tensor(loss, dtype=torch.float32), grad=grad)
    with qpg.Solver(*st["prob"], **_settings(case)) as s:  # instance
        g = st["net"].forward(s, case["rho"])
        D, E, c = s.scaling()
    return dict(g=g, D=D, E=E, c=c)


def _sizes(case):
    """Variables, constraints, entries of P and of A (expected values)."""
    f, a, b, dens = case["family"], case["a"], case["b"], case["dens"]
    if f == "control":
        T = case["t"]
        return (a * (T + 1) + b * T, a * (T + 1) + a * T + b * T, a * T + b * T + a,
                a * (2 * T + 1) + b * T + T * dens * (a * a + a * b))
    if f in ("random", "equality"):
        per = (min(dens, 4.47 / a) if dens < 0.15 else dens) * a
        return a, b, a * min(a, 1 + per * per), dens * a * b
    if f == "portfolio":
        return a + b, a + b + 1, a + b, dens * a * b + 2 * a + b
    if f == "svm":
        return a + b, 2 * a, b, dens * a * b + 2 * a
    return a + 2 * b, a + 2 * b, a, dens * a * b + a + 4 * b


#: ADMM iterations to the default tolerance and PCG steps of one solve, about as measured, by family.
_ITERS = dict(control=(2000, 2600), random=(120, 240), equality=(500, 520), lasso=(250, 500), svm=(60, 60))


def work(case):
    """The path's own traffic: each product reads its matrix once (value and index; P and both A and
    its transpose, the reduced KKT matrix being applied as P + sigma I + rho A^T A) and its vectors."""
    n, m, pe, ae = _sizes(case)
    s = 4 if case.get("mixed") else 8
    e = s + 4
    matvec = (pe + 2 * ae) * e + (14 * n + 2 * m) * s  # one PCG step
    flops = 2 * (pe + 2 * ae) + 12 * n
    kind = case["kind"]
    if kind in ("solve", "oneshot"):
        it, steps = _ITERS[case["family"]]
        rhs = (pe + ae) * e + 9 * n * s + 10 * m * s
        extra = 5 * (pe + 2 * ae) * 12 if kind == "oneshot" else 0
        return dict(bytes=float(steps * matvec + it * rhs + extra),
                    flops=float(steps * flops + it * (2 * (pe + ae) + 8 * m)))
    if kind == "pcg":
        steps = 45 if case["learned"] else 240 if case["family"] == "portfolio" else 60
        return dict(bytes=float(steps * matvec), flops=float(steps * flops))
    if kind == "hutchinson":
        # the matrix once per step for all probes together, the vectors once per probe
        steps = 120
        return dict(bytes=float(steps * ((pe + 2 * ae) * e + case["probes"] * (14 * n + 2 * m) * s)),
                    flops=float(steps * case["probes"] * flops))
    # forward: 3 rounds, each one product with A and one with its transpose on 32 features, and the
    # dense layers; backward twice that
    passes = 3 if kind == "train" else 1
    edges = 6 * ae * 8 + 8 * (n + m) * 32 * 4
    setup = 10 * (pe + 2 * ae) * 12 if kind == "instance" else 0
    return dict(bytes=float(passes * edges + setup), flops=float(passes * (6 * ae * 64 + 7 * (n + m) * 64 * 32)))


# ----------------------------------------------------- the same results in plain 64-bit arithmetic

class _Sparse:
    """Products with a matrix and its transpose in float64, by plain torch operations (as a dense
    matrix on the host where it is small)."""

    def __init__(self, M, dev):
        M = sp.csc_matrix(M)
        self.shape, self.dev = M.shape, dev
        self.r = torch.from_numpy(M.indices.astype(np.int64)).to(dev)
        self.ptr = torch.from_numpy(M.indptr.astype(np.int64)).to(dev)
        self.c = torch.repeat_interleave(torch.arange(M.shape[1], device=dev), self.ptr.diff())
        self.v = torch.from_numpy(M.data).to(dev)
        self._ops = None

    def scaled(self, rs, cs, f=1.0):
        self.v = self.v * rs[self.r] * cs[self.c] * f
        self._ops = None

    def _maxnorm(self, idx, count):
        return torch.zeros(count, device=self.dev, dtype=F64).scatter_reduce_(0, idx, self.v.abs(), "amax")

    def row_max(self):
        return self._maxnorm(self.r, self.shape[0])

    def col_max(self):
        return self._maxnorm(self.c, self.shape[1])

    def _csr(self):
        if self._ops is None and self.dev == "cpu":
            M = torch.zeros(self.shape, dtype=F64)
            M[self.r, self.c] = self.v
            self._ops = M, M.T
        if self._ops is None:
            order = torch.argsort(self.r * self.shape[1] + self.c)
            ptr = torch.zeros(self.shape[0] + 1, dtype=torch.int64, device=self.dev)
            ptr[1:] = torch.cumsum(torch.bincount(self.r, minlength=self.shape[0]), 0)
            self._ops = (torch.sparse_csr_tensor(ptr, self.c[order], self.v[order], size=self.shape),
                         torch.sparse_csr_tensor(self.ptr, self.r, self.v, size=self.shape[::-1]))
        return self._ops

    def mv(self, x):
        return self._csr()[0] @ x

    def tmv(self, x):
        return self._csr()[1] @ x

    def col_sq(self):
        return torch.zeros(self.shape[1], device=self.dev, dtype=F64).index_add_(0, self.c, self.v * self.v)


class _Scaled:
    """The equilibrated problem (modified Ruiz scaling, at most 10 passes) and its reduced KKT matrix."""

    SIGMA = 1e-6

    def __init__(self, prob):
        P_triu, q, A, lo, up = prob
        Pt = sp.csc_matrix(P_triu)
        n, m = A.shape[1], A.shape[0]
        self.dev = dev = "cpu" if n * (n + m) < 1_000_000 else "cuda"
        self.P = _Sparse(Pt + sp.triu(Pt, k=1).T, dev)
        self.A = _Sparse(A, dev)
        self.q0 = torch.from_numpy(np.asarray(q, np.float64)).to(dev)
        self.q = self.q0.clone()
        self.D = torch.ones(n, device=dev, dtype=F64)
        self.E = torch.ones(m, device=dev, dtype=F64)
        self.c = 1.0
        guard = lambda t: torch.where(t < 1e-4, torch.ones_like(t), t.clamp(max=1e4))  # noqa: E731
        for _ in range(10):
            d = guard(torch.maximum(self.P.col_max(), self.A.col_max())).rsqrt()
            e = guard(self.A.row_max()).rsqrt()
            self.D *= d
            self.E *= e
            self.P.scaled(d, d)
            self.A.scaled(e, d)
            self.q = self.q * d
            g = 1.0 / float(guard(torch.maximum(self.P.col_max().mean(), self.q.abs().max())))
            self.P.v = self.P.v * g
            self.q = self.q * g
            self.c *= g
            if max(float((1 - d).abs().max()), float((1 - e).abs().max()) if m else 0.0) <= 1e-3:
                break
        clamp = lambda t: torch.from_numpy(np.clip(np.asarray(t, np.float64), -1e20, 1e20)).to(dev)  # noqa: E731
        self.lo, self.up = self.E * clamp(lo), self.E * clamp(up)
        on = self.P.r == self.P.c
        self.diagP = torch.zeros(n, device=dev, dtype=F64).index_add_(0, self.P.r[on], self.P.v[on])
        self.colsq = self.A.col_sq()

    def K(self, x, rho):
        return self.P.mv(x) + self.SIGMA * x + self.A.tmv(rho * self.A.mv(x))

    def kdiag(self, rho):
        return self.diagP + self.SIGMA + rho * self.colsq

    def pcg(self, b, x, rho, minv, thresh, cap):
        r = self.K(x, rho) - b
        p = -minv * r
        rz = torch.dot(r, minv * r)
        it = 0
        while it < cap and float(r.abs().max()) > thresh:
            Kp = self.K(p, rho)
            alpha = rz / torch.dot(p, Kp)
            x = x + alpha * p
            r = r + alpha * Kp
            new = torch.dot(r, minv * r)
            p = -minv * r + (new / rz) * p
            rz = new
            it += 1
        return x, it


def _admm64(S):
    """The ADMM iteration with the inexact PCG step, default settings, in float64."""
    n, m = S.A.shape[1], S.A.shape[0]
    z64 = lambda k: torch.zeros(k, device=S.dev, dtype=F64)  # noqa: E731
    x, xt, z, y = z64(n), z64(n), z64(m), z64(m)
    rho, eps, alpha, lam = 0.1, 0.15, 1.6, 0.15
    best, since, tighten = INF, 0, 1.0
    amax = lambda t: float(t.abs().max()) if t.numel() else 0.0  # noqa: E731
    qn, qbn = amax(S.q0), amax(S.q)
    for k in range(1, 12_001 if S.dev == "cpu" else 3001):
        b = S.SIGMA * x - S.q + S.A.tmv(rho * z - y)
        xt, _ = S.pcg(b, xt, rho, 1.0 / S.kdiag(rho), eps * amax(b), 100)
        v = alpha * S.A.mv(xt) + (1 - alpha) * z
        z = torch.minimum(torch.maximum(v + y / rho, S.lo), S.up)
        y = y + rho * (v - z)
        x = alpha * xt + (1 - alpha) * x
        if k % 5:
            continue
        Ax, Px, Aty = S.A.mv(x), S.P.mv(x), S.A.tmv(y)
        rp, rd = Ax - z, Px + S.q + Aty
        prim, dual = amax(rp / S.E), amax(rd / S.D) / S.c
        ep = 1e-3 + 1e-3 * max(amax(Ax / S.E), amax(z / S.E))
        ed = 1e-3 + 1e-3 * max(amax(Px / S.D) / S.c, amax(Aty / S.D) / S.c, qn)
        if prim <= ep and dual <= ed:
            return S.D * x, S.E * y / S.c, k
        ratio = max(prim / ep, dual / ed)
        if ratio < 0.99 * best:
            best, since = ratio, 0
        else:
            since += 1
        if since >= 10 and since % 2 == 0:
            tighten = max(0.1 * tighten, 1e-12)
        np_, nd = amax(rp), amax(rd)
        eps = max(min(lam * math.sqrt(np_ * nd), lam) * tighten, 1e-7)
        if k % 10 == 0:
            num = np_ / max(amax(Ax), amax(z), 1e-10)
            den = nd / max(amax(Px), amax(Aty), qbn, 1e-10)
            if num > 0 and den > 0:
                rho = min(max(rho * math.sqrt(num / den), 1e-6), 1e6)
    return None


class _Net64:
    """The message-passing network in float64; dense weights rounded to bfloat16, as the network
    stores them for its matrix products."""

    H, L = 32, 3

    def __init__(self, flat, dev):
        t = torch.from_numpy(np.asarray(flat, np.float64)).to(dev).requires_grad_(True)
        self.flat, o = t, 0

        def take(*shape):
            nonlocal o
            k = math.prod(shape)
            w = t[o:o + k].reshape(shape)
            o += k
            return w

        def layer(k):
            w, b = take(k, self.H), take(self.H)
            return w + (w.detach().float().bfloat16().to(F64) - w.detach()), b

        self.v0, self.c0 = layer(32), layer(32)
        self.rounds = [(layer(64), layer(64)) for _ in range(self.L)]
        self.h1 = layer(64)
        self.w2, self.b2 = take(self.H), take(1)

    def forward(self, S, rho):
        n, m = S.A.shape[1], S.A.shape[0]
        r, c, w = S.A.r, S.A.c, S.A.v.abs()
        z = lambda k: torch.zeros(k, device=S.dev, dtype=F64)  # noqa: E731
        rs, cs = z(m).index_add_(0, r, w), z(n).index_add_(0, c, w)
        hat, chk = w / rs[r], w / cs[c]
        deg_r, deg_c = torch.bincount(r, minlength=m).to(F64), torch.bincount(c, minlength=n).to(F64)
        pad = lambda cols, k: torch.cat([torch.stack(cols, 1), z(k * (self.H - len(cols))).reshape(k, -1)], 1)  # noqa: E731
        K = S.kdiag(rho)
        fv = pad([(S.diagP + S.SIGMA).log(), (S.colsq + 1e-12).log(), deg_c.log1p(), (S.A.col_max() + 1e-12).log()], n)
        fc = pad([(z(m).index_add_(0, r, w * w) + 1e-12).log(), deg_r.log1p(), (S.lo == S.up).to(F64),
                  (S.A.row_max() + 1e-12).log()], m)
        phi = pad([(rho * S.colsq + 1e-12).log() - K.log(), (S.diagP + S.SIGMA).log() - K.log()], n)
        dense = lambda X, wb: torch.relu(X @ wb[0] + wb[1])  # noqa: E731
        spmm = lambda w, to, frm, X, k: torch.zeros(k, self.H, device=S.dev, dtype=F64).index_add(0, to, w[:, None] * X[frm])  # noqa: E731
        hv, hc = dense(fv, self.v0), dense(fc, self.c0)
        for wc, wv in self.rounds:
            hc = dense(torch.cat([hc, spmm(hat, r, c, hv, m)], 1), wc)
            hv = dense(torch.cat([hv, spmm(chk, c, r, hc, n)], 1), wv)
        return dense(torch.cat([hv, phi], 1), self.h1) @ self.w2 + self.b2


def exact(case, seed):
    kind = case["kind"]
    prob = _problem(case, seed)
    rng = np.random.default_rng(seed)
    S = _Scaled(prob)
    n = prob[2].shape[1]
    if kind in ("solve", "oneshot"):
        got = _admm64(S)
        if got is None:
            return None
        return dict(x=got[0].cpu(), y=got[1].cpu(), iters=None)
    if kind == "pcg":
        b = torch.from_numpy(rng.standard_normal(n)).to(S.dev)
        minv = 1.0 / S.kdiag(case["rho"])
        x, _ = S.pcg(b, torch.zeros_like(b), case["rho"], minv, 1e-14 * float(b.abs().max()), 1500)
        return dict(x=x.cpu(), iters=None)
    if kind == "hutchinson":
        signs = rng.choice(np.array([-1, 1], dtype=np.int8), size=(case["probes"], n))
        acc = torch.zeros(n, device=S.dev, dtype=F64)
        minv = 1.0 / S.kdiag(case["rho"])
        for row in signs:
            zk = torch.from_numpy(row.astype(np.float64)).to(S.dev)
            acc += zk * S.pcg(zk, torch.zeros_like(zk), case["rho"], minv, 1e-14, 500)[0]
        return dict(diag=(acc / len(signs)).cpu())
    net = _Net64(_weights(case), S.dev)
    if kind == "instance":
        with torch.no_grad():
            g = net.forward(S, case["rho"])
        return dict(g=g.cpu(), D=S.D.cpu(), E=S.E.cpu(), c=S.c)
    target = torch.from_numpy(np.abs(rng.normal(0.0, 0.5, n)).astype(np.float32)).to(S.dev).to(F64)
    g = net.forward(S, case["rho"])
    e = torch.log(torch.nn.functional.softplus(g)) - target
    loss = ((e - e.mean()) ** 2).mean()
    loss.backward()
    return dict(loss=loss.detach().cpu(), grad=net.flat.grad.cpu())
