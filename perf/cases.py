"""What a user of this library has it do, as a list of measurable cases.

listed() / draw(rng) name the work, prepare() makes what a program holds before the call (inputs on
the GPU, a context, the problem, the stages it keeps), run() makes one pass through the public entry
points and exact() gives the same outputs in 64 bits from plain torch / numpy.

Kinds of case
  call          bbmm_solve_logdet_grad: one optimiser step on hyperparameters (solve, log-det, gradient)
  mm            bbmm_kernel_mm: the product K_hat M on its own
  predict_mean  posterior means at a batch of test inputs
  predict_var   posterior variances at up to 32 test inputs (one more preconditioned mBCG run)
  dk            bbmm_dk_traces: all derivative terms for given solves
  precond       preconditioner from scratch, the probes and one solve with it
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1809_11165_amd import binding, inputs

MODES = {"mat": inputs.MATERIALISED, "sym": inputs.MATERIALISED, "otf": inputs.ONTHEFLY, "sgpr": inputs.SGPR}


def listed():
    return [
        # a training step on a small tabular set with the settings of the paper's regression runs
        # (rank-5 preconditioner, 10 probes, 20 iterations): latency and launches decide
        {"name": "train_small", "kind": "call", "recipe": 1, "mode": "mat", "n": 1000, "t": 10, "k": 5, "iters": 20},
        # a medium set run to convergence, the whole matrix kept
        {"name": "train_medium", "kind": "call", "recipe": 2, "mode": "mat", "n": 10000, "t": 10, "k": 10, "iters": 160},
        # the benchmark problem at its converged iteration cap, upper triangle kept
        {"name": "train_large_triangle", "kind": "call", "recipe": 3, "mode": "sym", "n": 50000, "t": 10, "k": 20, "iters": 100},
        # the same recipe without ever storing the matrix, odd size
        {"name": "train_large_onthefly", "kind": "call", "recipe": 3, "mode": "otf", "n": 30011, "t": 10, "k": 20, "iters": 100},
        # sparse GP step: half a million points, 1024 inducing inputs
        {"name": "train_sparse", "kind": "call", "recipe": 5, "mode": "sgpr", "n": 500000, "t": 10, "k": 10, "iters": 128,
         "m": 1024},
        # the product of the largest exact workload: 16 probes and y, matrix too large to want to store
        {"name": "product_huge_onthefly", "kind": "mm", "recipe": 4, "mode": "otf", "n": 200000, "c": 17},
        # the product on a small stored matrix
        {"name": "product_small", "kind": "mm", "recipe": 2, "mode": "mat", "n": 5000, "c": 11},
        # serving: variances of a full batch of 32 test points
        {"name": "variance_batch", "kind": "predict_var", "recipe": 3, "mode": "mat", "n": 20000, "k": 20, "iters": 60, "ns": 32},
        # serving: means of a batch of test points, and of a single one (latency)
        {"name": "mean_batch", "kind": "predict_mean", "recipe": 3, "mode": "otf", "n": 50000, "ns": 1024},
        {"name": "mean_single", "kind": "predict_mean", "recipe": 3, "mode": "otf", "n": 50000, "ns": 1},
        # all d + 2 derivative terms of a large ARD problem for solves in hand
        {"name": "derivative_terms", "kind": "dk", "recipe": 3, "mode": "otf", "n": 50000, "t": 10},
        # a new preconditioner after a hyperparameter change
        {"name": "preconditioner", "kind": "precond", "recipe": 3, "mode": "otf", "n": 50000, "t": 10, "k": 20},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["call", "call", "call", "mm", "mm", "predict_mean", "predict_var", "dk", "precond"])
    t = rng.choice([1, 4, 8, 10, 10, 11, 12, 15, 16, 20, 31])
    k = rng.choice([0, 2, 5, 9, 10, 15, 20, 31])
    if kind == "call":
        mode = rng.choice(["mat", "sym", "otf", "otf", "sgpr"])
        if mode == "sgpr":
            return {"kind": kind, "recipe": 5, "mode": mode, "n": _log_int(rng, 3000, 400000), "t": min(t, 20), "k": max(k, 2),
                    "iters": 128, "m": _log_int(rng, 40, 1024)}
        recipe = rng.choice([1, 2, 3])
        top = {1: 4000, 2: 15000, 3: 40000}[recipe]
        return {"kind": kind, "recipe": recipe, "mode": mode, "n": _log_int(rng, 500, top), "t": t, "k": max(k, 5),
                "iters": {1: 20, 2: 160, 3: 100}[recipe]}
    if kind == "mm":
        mode = rng.choice(["mat", "sym", "otf", "otf"])
        return {"kind": kind, "recipe": rng.choice([1, 2, 3, 4]), "mode": mode,
                "n": _log_int(rng, 700, 150000 if mode == "otf" else 60000), "c": rng.randint(1, 32)}
    if kind == "predict_mean":
        return {"kind": kind, "recipe": rng.choice([1, 2, 3, 4]), "mode": "otf", "n": _log_int(rng, 1000, 80000),
                "ns": _log_int(rng, 1, 2000)}
    if kind == "predict_var":
        return {"kind": kind, "recipe": 3, "mode": rng.choice(["mat", "otf"]), "n": _log_int(rng, 1000, 20000), "k": max(k, 2),
                "iters": 60, "ns": rng.randint(1, 32)}
    if kind == "dk":
        return {"kind": kind, "recipe": rng.choice([1, 2, 3]), "mode": "otf", "n": _log_int(rng, 1000, 50000), "t": t}
    return {"kind": kind, "recipe": rng.choice([1, 2, 3]), "mode": "otf", "n": _log_int(rng, 1000, 80000), "t": t, "k": max(k, 2)}


# ------------------------------------------------------------------------------- inputs
def _workload(case, seed):
    """The repository's synthetic recipe at this size; the seed picks independent inputs."""
    kw = {"n": case["n"], "t": case.get("t", 1), "k": case.get("k", 0), "iters": case.get("iters", 1), "salt": 1 + seed}
    if case["recipe"] == 5:
        kw["m"] = case["m"]
    w = inputs.make(case["recipe"], **kw)
    w.tol = 0.0
    if case["recipe"] == 5:
        # enough noise for 128 iterations to resolve the solves (at 0.01 they end unconverged, where
        # two correct summation orders already differ by percents)
        w.noise = 0.25
    return w


def _rng(case, seed, salt):
    return np.random.Generator(np.random.Philox(np.random.SeedSequence([77, seed, salt])))


def _normal(case, seed, salt, shape):
    a = _rng(case, seed, salt).standard_normal(shape, dtype=np.float32)
    return torch.from_numpy(a).cuda()


def _test_inputs(case, seed, w):
    """Test inputs from the training distribution: a training point moved by a fifth of the spread."""
    r = _rng(case, seed, 5)
    rows = r.integers(0, w.n, size=case["ns"])
    xs = w.X[rows] + 0.2 * w.X.std(axis=0) * r.standard_normal((case["ns"], w.d))
    return torch.from_numpy(np.ascontiguousarray(xs, dtype=np.float32)).cuda()


def _pivots(w):
    """Sparse problems replay a pivot order (the greedy one is not unique there): the first inducing rows."""
    return np.ascontiguousarray(w.meta["inducing_rows"][:w.k], dtype=np.int64)


def prepare(case, seed):
    w = _workload(case, seed)
    mode = MODES[case["mode"]]
    ctx = binding.Context(0)
    if case["mode"] == "sym":
        ctx.bbmm_tune("khat_sym", 1)
    prob = binding.problem_from_workload(w, mode)
    if case["mode"] == "sgpr":
        prob.pivots_in = _pivots(w)
    st = {"case": case, "ctx": ctx, "prob": prob, "mode": mode}
    kind = case["kind"]
    if kind == "call":
        return st
    ctx.bbmm_setup(prob)
    if kind == "mm":
        if mode == inputs.MATERIALISED:
            ctx.bbmm_build_khat()
        st["M"] = _normal(case, seed, 1, (w.n, case["c"]))
    elif kind == "predict_mean":
        st["u0"] = _normal(case, seed, 2, (w.n,))
        st["Xstar"] = _test_inputs(case, seed, w)
    elif kind == "predict_var":
        if mode == inputs.MATERIALISED:
            ctx.bbmm_build_khat()
        ctx.bbmm_pivoted_cholesky()
        ctx.bbmm_precond_setup()
        st["Xstar"] = _test_inputs(case, seed, w)
    elif kind == "dk":
        st["U"] = _normal(case, seed, 3, (w.n, w.t + 1))
        st["W"] = _normal(case, seed, 4, (w.n, w.t))
    elif kind == "precond":
        st["R"] = _normal(case, seed, 6, (w.n, w.t + 1))
    return st


def run(st):
    ctx, kind = st["ctx"], st["case"]["kind"]
    if kind == "call":
        r = ctx.bbmm_solve_logdet_grad(st["prob"])
        return {"u0": r.u0, "U": r.U, "logdet": r.logdet, "logdet_precond": r.logdet_precond, "yKinvy": r.yKinvy, "nlml": r.nlml,
                "trace": r.trace, "quad": r.quad, "grad": r.grad_nlml, "slq_terms": r.slq_terms}
    if kind == "mm":
        return ctx.bbmm_kernel_mm(st["mode"], st["M"])
    if kind == "predict_mean":
        return ctx.bbmm_predict_mean(st["Xstar"], st["u0"])
    if kind == "predict_var":
        return ctx.bbmm_predict_var(st["mode"], st["Xstar"])[0]
    if kind == "dk":
        trace, quad = ctx.bbmm_dk_traces(st["U"], st["W"])
        return {"trace": trace, "quad": quad}
    L, piv, _ = ctx.bbmm_pivoted_cholesky()
    logdet_p = ctx.bbmm_precond_setup()
    return {"L": L, "pivots": piv, "logdet_precond": logdet_p, "probes": ctx.bbmm_make_probes(),
            "solve": ctx.bbmm_precond_solve(st["R"])}


_DIM = {1: 4, 2: 8, 3: 16, 4: 8, 5: 8}


def work(case):
    """Inputs once, outputs once; one multiplication and one addition per term of each contraction and
    about ten operations per kernel value."""
    n, d, kind = case["n"], _DIM[case["recipe"]], case["kind"]
    kernel = 2.0 * d + 10.0
    if kind == "mm":
        c = case["c"]
        stored = {"mat": 4.0 * n * n, "sym": 2.0 * n * n, "otf": 4.0 * n * d}[case["mode"]]
        return {"bytes": stored + 8.0 * n * c, "flops": n * n * (2.0 * c + (kernel if case["mode"] == "otf" else 0.0))}
    if kind == "predict_mean":
        ns = case["ns"]
        return {"bytes": 4.0 * (n * d + ns * d + n + ns), "flops": n * ns * (kernel + 2.0)}
    if kind == "dk":
        t = case["t"]
        per = 2.0 * 2 * t + kernel + (8.0 * d if case["recipe"] == 3 else 8.0)
        return {"bytes": 4.0 * n * (d + 2 * t + 1), "flops": 0.5 * n * n * per}
    if kind == "precond":
        t, k = case["t"], case["k"]
        return {"bytes": 4.0 * n * (d + 3 * t + 4) + 8.0 * n * k,
                "flops": n * k * (kernel + k) + 2.0 * n * k * k + n * k * (2.0 * t + 4.0 * (t + 1))}
    iters, k = case["iters"], case["k"]
    if kind == "predict_var":
        ns = case["ns"]
        stored = 4.0 * n * n if case["mode"] == "mat" else 4.0 * n * d
        per = 2.0 * ns + (kernel if case["mode"] == "otf" else 0.0)
        return {"bytes": stored + 4.0 * ns, "flops": iters * (n * n * per + 4.0 * n * k * ns) + 2.0 * n * ns * kernel}
    t = case["t"]
    c = t + 1
    io = 4.0 * n * (d + 1 + t + 1 + c) + 4.0 * k * t
    if case["mode"] == "sgpr":
        m = case["m"]
        return {"bytes": io + 4.0 * m * d,
                "flops": n * m * (kernel + m) + iters * (4.0 * n * m * c + 4.0 * n * k * c) + 2.0 * n * m * k + n * m * (4.0 * t + 8.0 * d)}
    evals = iters if case["mode"] == "otf" else 1
    deriv = 0.5 * n * n * (4.0 * t + kernel + (8.0 * d if case["recipe"] == 3 else 8.0))
    return {"bytes": io, "flops": iters * (2.0 * n * n * c + 4.0 * n * k * c) + evals * 0.5 * n * n * kernel + deriv}


def tolerance(case):
    """Matrix entries and block outputs are 32-bit.  About four times the distance from the 64-bit
    values that the path itself shows at these sizes, which for the iterative cases is the rounding of
    the entries times the conditioning of the system."""
    kind = case["kind"]
    if kind == "call":
        if case["mode"] == "sgpr":
            return {"rel": 2e-4}
        return {"rel": {1: 1e-4, 2: 1e-4, 3: 4e-5}[case["recipe"]]}
    return {"rel": {"mm": 4e-6, "predict_mean": 1e-6, "predict_var": 1e-5, "dk": 5e-5, "precond": 1e-6}[kind]}


# ----------------------------------------------------------------- the same in 64 bits
def _k64(kernel, Xa, Xb, ls, s):
    """(k, g): kernel values and the radial weight of the lengthscale derivative, both times s."""
    a, b = Xa / ls, Xb / ls
    r2 = (a * a).sum(1)[:, None] + (b * b).sum(1)[None, :] - 2.0 * (a @ b.T)
    r2.clamp_(min=0.0)
    if kernel == inputs.RBF:
        k = torch.exp(r2.mul_(-0.5)).mul_(s)
        return k, k
    rho = r2.sqrt().mul_(math.sqrt(5.0))
    e = torch.exp(-rho).mul_(s)
    g = (1.0 + rho).mul_(e).mul_(5.0 / 3.0)
    k = r2.mul_(5.0 / 3.0).add_(rho).add_(1.0).mul_(e)
    return k, g


def _row_exact(kernel, X, i, ls, s):
    df = (X - X[i]) / ls
    r2 = (df * df).sum(1)
    if kernel == inputs.RBF:
        return s * torch.exp(-0.5 * r2)
    rho = r2.sqrt()
    s5 = math.sqrt(5.0)
    return s * (1.0 + s5 * rho + (5.0 / 3.0) * r2) * torch.exp(-s5 * rho)


class _Dense:
    """K_XX, held or in row chunks, in 64 bits."""

    def __init__(self, w, X, hold):
        self.w, self.X = w, X
        self.ls = torch.from_numpy(np.broadcast_to(w.lengthscale, (w.d,)).copy()).cuda()
        self.step = max(64, min(w.n, int(2.5e8 // w.n)))
        self.held = None
        if hold:
            self.held = torch.empty(w.n, w.n, dtype=torch.float64, device="cuda")
            for i, j, k, _ in self.chunks():
                self.held[i:j] = k

    def chunks(self):
        n = self.w.n
        for i in range(0, n, self.step):
            j = min(n, i + self.step)
            k, g = _k64(self.w.kernel, self.X[i:j], self.X, self.ls, self.w.outputscale)
            k[torch.arange(j - i), torch.arange(i, j)] = self.w.outputscale
            yield i, j, k, g

    def mm(self, D):
        if self.held is not None:
            return self.held @ D
        return torch.cat([k @ D for _, _, k, _ in self.chunks()])

    def diag(self):
        return torch.full((self.w.n,), self.w.outputscale, dtype=torch.float64, device="cuda")

    def row(self, i):
        return _row_exact(self.w.kernel, self.X, i, self.ls, self.w.outputscale)

    def derivative_sums(self, A, B):
        """sum_ij (dK/dtheta_h)_ij sum_q A_iq B_jq for the lengthscale(s) and the outputscale."""
        w = self.w
        Xl = self.X / self.ls
        per = torch.zeros(w.d, dtype=torch.float64, device="cuda")
        es = 0.0
        for i, j, k, g in self.chunks():
            S = A[i:j] @ B.T
            es += float((k * S).sum()) / w.outputscale
            T = S.mul_(g)
            del k, g
            xi = Xl[i:j]
            per += (xi * xi * T.sum(1)[:, None]).sum(0) + (Xl * Xl * T.sum(0)[:, None]).sum(0) - 2.0 * (xi * (T @ Xl)).sum(0)
        if len(w.lengthscale) == 1:
            return np.array([float(per.sum()) / w.lengthscale[0], es])
        return np.concatenate([(per / self.ls).cpu().numpy(), [es]])


class _Sparse:
    """Q = K_XU (K_UU + jitter)^-1 K_UX through its root, in 64 bits."""

    def __init__(self, w, X):
        self.w, self.X = w, X
        self.ls = torch.from_numpy(np.broadcast_to(w.lengthscale, (w.d,)).copy()).cuda()
        self.U = torch.from_numpy(w.Uind.astype(np.float64)).cuda()
        m = self.U.shape[0]
        kuu, self.guu = _k64(w.kernel, self.U, self.U, self.ls, w.outputscale)
        self.kuu = kuu.clone()
        self.kuu[torch.arange(m), torch.arange(m)] = w.outputscale
        jit = self.kuu + w.jitter_rel * w.outputscale * torch.eye(m, dtype=torch.float64, device="cuda")
        self.G = torch.linalg.cholesky(jit)
        kxu, self.gxu = _k64(w.kernel, self.X, self.U, self.ls, w.outputscale)
        ginv = torch.linalg.solve_triangular(self.G, torch.eye(m, dtype=torch.float64, device="cuda"), upper=False)
        self.A = kxu @ ginv.T.contiguous()

    def mm(self, D):
        return self.A @ (self.A.T @ D)

    def diag(self):
        return (self.A * self.A).sum(1)

    def row(self, i):
        return self.A @ self.A[i]

    def _pairs(self, g, Xa, Xb, P, Q):
        T = g * (P @ Q.T)
        return (Xa * Xa * T.sum(1)[:, None]).sum(0) + (Xb * Xb * T.sum(0)[:, None]).sum(0) - 2.0 * (Xa * (T @ Xb)).sum(0)

    def derivative_sums(self, A, B):
        w = self.w
        ta, tb = self.A.T @ A, self.A.T @ B
        ba = torch.linalg.solve_triangular(self.G.T, ta, upper=True)
        bb = torch.linalg.solve_triangular(self.G.T, tb, upper=True)
        Xl, Ul = self.X / self.ls, self.U / self.ls
        per = self._pairs(self.gxu, Xl, Ul, A, bb) + self._pairs(self.gxu, Xl, Ul, B, ba) - self._pairs(self.guu, Ul, Ul, ba, bb)
        es = float((ta * tb).sum()) / w.outputscale
        if len(w.lengthscale) == 1:
            return np.array([float(per.sum()) / w.lengthscale[0], es])
        return np.concatenate([(per / self.ls).cpu().numpy(), [es]])


def _pivoted_cholesky64(op, n, k, forced=None):
    L = torch.zeros(n, k, dtype=torch.float64, device="cuda")
    delta = op.diag().clone()
    piv = []
    for m in range(k):
        p = int(forced[m]) if forced is not None else int(delta.argmax())
        if forced is None:
            p = int((delta == delta[p]).nonzero()[0, 0])
        root = torch.sqrt(delta[p])
        col = (op.row(p) - L[:, :m] @ L[p, :m]) / root
        if piv:
            col[torch.tensor(piv, device="cuda")] = 0.0
        col[p] = root
        L[:, m] = col
        delta = (delta - col * col).clamp(min=0.0)
        piv.append(p)
        delta[torch.tensor(piv, device="cuda")] = -1.0
    return L, piv


class _Precond:
    def __init__(self, L, noise):
        self.L, self.noise = L, noise
        n, k = L.shape
        C = noise * torch.eye(k, dtype=torch.float64, device="cuda") + L.T @ L
        self.chol = torch.linalg.cholesky(C) if k else C
        self.logdet = (2.0 * float(torch.log(torch.diagonal(self.chol)).sum()) if k else 0.0) + (n - k) * math.log(noise)

    def solve(self, R):
        if self.L.shape[1] == 0:
            return R / self.noise
        return (R - self.L @ torch.cholesky_solve(self.L.T @ R, self.chol)) / self.noise


def _mbcg64(op, P, noise, B, iters):
    U, R = torch.zeros_like(B), B.clone()
    Z = P.solve(R)
    Z0, D = Z.clone(), Z.clone()
    rho = (R * Z).sum(0)
    rho0 = rho.clone()
    alphas, betas = [], []
    for _ in range(iters):
        V = op.mm(D) + noise * D
        a = rho / (D * V).sum(0)
        U += a * D
        R -= a * V
        Z = P.solve(R)
        new = (R * Z).sum(0)
        b = new / rho
        D = Z + b * D
        rho = new
        alphas.append(a)
        betas.append(b)
    return U, Z0, rho0, torch.stack(alphas).cpu().numpy(), torch.stack(betas).cpu().numpy()


def _slq64(alpha, beta, rho0):
    from scipy.linalg import eigh_tridiagonal
    terms = []
    for q in range(alpha.shape[1]):
        a, b = alpha[:, q], beta[:, q]
        dg = 1.0 / a
        dg[1:] += b[:-1] / a[:-1]
        off = np.sqrt(b[:-1]) / a[:-1]
        lam, vec = eigh_tridiagonal(dg, off, lapack_driver="stev")
        terms.append(rho0[q] * float(np.sum(vec[0] ** 2 * np.log(np.maximum(lam, 1e-300)))))
    return np.array(terms)


def exact(case, seed):
    w = _workload(case, seed)
    X = torch.from_numpy(w.X.astype(np.float64)).cuda()
    kind = case["kind"]
    if kind == "mm":
        op = _Dense(w, X, False)
        M = _normal(case, seed, 1, (w.n, case["c"])).double()
        return op.mm(M) + w.noise * M
    if kind == "predict_mean":
        ls = torch.from_numpy(np.broadcast_to(w.lengthscale, (w.d,)).copy()).cuda()
        u0 = _normal(case, seed, 2, (w.n,)).double()
        xs = _test_inputs(case, seed, w).double()
        step = max(1, int(2e8 // w.n))
        return torch.cat([_k64(w.kernel, xs[a:a + step], X, ls, w.outputscale)[0] @ u0 for a in range(0, xs.shape[0], step)])
    if kind == "dk":
        op = _Dense(w, X, False)
        U = _normal(case, seed, 3, (w.n, w.t + 1)).double()
        W = _normal(case, seed, 4, (w.n, w.t)).double()
        trace = np.append(op.derivative_sums(U[:, 1:], W), float((U[:, 1:] * W).sum())) / w.t
        quad = np.append(op.derivative_sums(U[:, :1], U[:, :1]), float((U[:, 0] ** 2).sum()))
        return {"trace": trace, "quad": quad}
    sparse = case["mode"] == "sgpr"
    op = _Sparse(w, X) if sparse else _Dense(w, X, hold=kind != "precond")
    L, piv = _pivoted_cholesky64(op, w.n, w.k, _pivots(w) if sparse else None)
    P = _Precond(L, w.noise)
    if kind == "predict_var":
        xs = _test_inputs(case, seed, w).double()
        B = _k64(w.kernel, X, xs, op.ls, w.outputscale)[0]
        U = _mbcg64(op, P, w.noise, B, w.iters)[0]
        return w.outputscale - (B * U).sum(0)
    E1, E2 = torch.from_numpy(w.E1).cuda().double(), torch.from_numpy(w.E2).cuda().double()
    y = torch.from_numpy(w.y).cuda().double()
    B = torch.cat([y[:, None], L @ E1 + math.sqrt(w.noise) * E2], 1)
    if kind == "precond":
        R = _normal(case, seed, 6, (w.n, w.t + 1)).double()
        return {"L": L, "pivots": None, "logdet_precond": P.logdet, "probes": B, "solve": P.solve(R)}
    U, Z0, rho0, alpha, beta = _mbcg64(op, P, w.noise, B, w.iters)
    terms = _slq64(alpha[:, 1:].copy(), beta[:, 1:].copy(), rho0[1:].cpu().numpy())
    trace = np.append(op.derivative_sums(U[:, 1:], Z0[:, 1:]), float((U[:, 1:] * Z0[:, 1:]).sum())) / w.t
    quad = np.append(op.derivative_sums(U[:, :1], U[:, :1]), float((U[:, 0] ** 2).sum()))
    logdet = P.logdet + float(terms.mean())
    ykiy = float((y * U[:, 0]).sum())
    return {"u0": U[:, 0], "U": U, "logdet": logdet, "logdet_precond": P.logdet, "yKinvy": ykiy,
            "nlml": 0.5 * (ykiy + logdet + w.n * math.log(2.0 * math.pi)), "trace": trace, "quad": quad,
            "grad": 0.5 * (trace - quad), "slq_terms": terms}
