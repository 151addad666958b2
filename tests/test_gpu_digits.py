"""GPU: the on-the-fly product on the 8-bit matrix pipe (at most 16 input dimensions, from 6144 padded rows
on) against fp64 kernel rows, over block widths, dimensions and sizes at the edges of its tiles."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import bbmm_oracle as O  # noqa: E402
from paper_1809_11165_amd import inputs  # noqa: E402

N0 = 6144            # first size of the route; 16-row tiles, workgroups of 4 * (2 .. 6) tiles, pads of 256


@pytest.fixture(scope="module")
def ctx():
    from paper_1809_11165_amd import binding
    c = binding.Context(0)
    c.bbmm_tune("otf_digits", 2)         # whatever the block
    yield c
    c.close()


def _problem(n, d, kernel, X=None, noise=0.1):
    from paper_1809_11165_amd import binding
    w = inputs.tiny(n, d, kernel=kernel, ard=d > 1, t=1, k=1, iters=1, noise=noise, seed=3)
    if X is not None:
        w.X = X.astype(np.float32)
    return w, binding.problem_from_workload(w, inputs.ONTHEFLY)


def _rows(w, rows, M):
    """Rows of K_hat M in fp64 and the bound on their error.

    The squared distance is formed in fp32 from |x|^2 + |x'|^2 - 2 x.x' of scaled, centred coordinates rounded to
    fp32: every one of its roundings is at most 2^-24 of |x|^2 + |x'|^2, and four of them are allowed for (two
    squared norms, the product, the last addition; longer sums round at random).  The entry moves by what the
    kernel function makes of that, by 2^-22 of itself in its own evaluation, and by half a unit of the
    fixed-point scale; the sum over the row is bounded term by term.  The result is rounded to fp32."""
    X = w.X.astype(np.float64)
    K = O.kernel_block(w.kernel, X[rows], X, w.lengthscale, w.outputscale)
    xs = (X - X.mean(axis=0)) / w.lengthscale
    sq = (xs * xs).sum(axis=1)
    r2 = np.maximum(sq[rows][:, None] + sq[None, :] - 2.0 * xs[rows] @ xs.T, 0.0)
    delta = 4 * 2.0 ** -24 * (sq[rows][:, None] + sq[None, :])

    def k(r2):
        if w.kernel == inputs.RBF:
            return w.outputscale * np.exp(-0.5 * r2)
        a = np.sqrt(5.0 * r2)
        return w.outputscale * (1.0 + a + a * a / 3.0) * np.exp(-a)

    dK = k(np.maximum(r2 - delta, 0.0)) - k(r2 + delta) + 2.0 ** -22 * K + 0.5 * w.outputscale / 2055208960.0
    dK[np.arange(len(rows)), rows] = 2.0 ** -22 * w.outputscale
    K[np.arange(len(rows)), rows] = w.outputscale + w.noise
    ref = K @ M
    return ref, dK @ np.abs(M) + 2.0 ** -23 * np.abs(ref)


def _check(V, ref, bound):
    err = np.abs(V - ref)
    assert np.all(err <= bound), float((err / np.maximum(bound, 1e-300)).max())


@pytest.mark.parametrize("kernel", [inputs.RBF, inputs.MATERN52])
@pytest.mark.parametrize("n,d,c", [(N0, 1, 1), (N0 + 1, 3, 4), (N0 - 100, 4, 5), (6400, 4, 8), (6401, 5, 9), (7000, 8, 12),
                                   (6999, 8, 13), (6656, 9, 16), (6657, 16, 17), (7169, 16, 18), (6300, 2, 19),
                                   (6200, 13, 24), (6500, 7, 25), (6911, 16, 32), (9000, 16, 11), (8193, 4, 32)])
def test_digit_product_against_fp64_rows(ctx, kernel, n, d, c):
    import torch
    w, prob = _problem(n, d, kernel)
    rng = np.random.default_rng(n + 31 * c)
    M = rng.standard_normal((n, c)).astype(np.float32)
    M[:, -1] *= 1e-25                                   # a scale of its own per column
    if c > 1:
        M[:, 0] = 1.0 + 0.1 * M[:, 0]                   # no cancellation
    if c > 2:
        M[:, 1] = 0.0
    if c > 3:
        M[:, 2] *= np.exp(3.0 * rng.standard_normal(n)) # one entry far above the others
    ctx.bbmm_setup(prob)
    V = ctx.bbmm_kernel_mm(inputs.ONTHEFLY, torch.from_numpy(M).cuda()).cpu().numpy().astype(np.float64)
    rows = np.unique(np.concatenate([[0, 15, 16, n - 1, n - 2, n // 2], rng.integers(0, n, 60)]))
    M64 = M.astype(np.float64)
    _check(V[rows], *_rows(w, rows, M64))
    if c > 2:
        assert not V[:, 1].any()


@pytest.mark.parametrize("kernel", [inputs.RBF, inputs.MATERN52])
def test_digit_product_with_near_duplicate_points(ctx, kernel):
    """Entries at and just below one (the largest digits)."""
    import torch
    n, d = 6300, 4
    rng = np.random.default_rng(5)
    X = rng.standard_normal((n, d))
    X[1::2] = X[0:n - 1:2] + 1e-3 * rng.standard_normal((n // 2, d)) * (rng.random((n // 2, 1)) < 0.5)
    w, prob = _problem(n, d, kernel, X=X)
    M = rng.standard_normal((n, 11)).astype(np.float32)
    ctx.bbmm_setup(prob)
    V = ctx.bbmm_kernel_mm(inputs.ONTHEFLY, torch.from_numpy(M).cuda()).cpu().numpy().astype(np.float64)
    rows = rng.integers(0, n, 80)
    M64 = M.astype(np.float64)
    _check(V[rows], *_rows(w, rows, M64))


def test_digit_product_of_non_finite_blocks(ctx):
    """A column with an infinity or a NaN gets what the fp64 form gives where no entry of K vanishes; the others are not
    touched.  (otf_digits = 1 takes the fp64 form for such a block.)"""
    import torch
    w, prob = _problem(6200, 4, inputs.RBF)
    M = np.random.default_rng(1).standard_normal((6200, 6)).astype(np.float32)
    M[7, 1], M[9, 2], M[11, 3] = np.inf, -np.inf, np.nan
    M[3, 4], M[4, 4] = np.inf, -np.inf
    Md = torch.from_numpy(M).cuda()
    ctx.bbmm_setup(prob)
    V = ctx.bbmm_kernel_mm(inputs.ONTHEFLY, Md).cpu().numpy()
    ctx.bbmm_tune("otf_sym", 0)
    try:
        ref = ctx.bbmm_kernel_mm(inputs.ONTHEFLY, Md).cpu().numpy()
    finally:
        ctx.bbmm_tune("otf_sym", 1)
    np.testing.assert_allclose(V[:, [0, 5]], ref[:, [0, 5]], rtol=0, atol=2e-6 * np.abs(ref[:, [0, 5]]).max())
    np.testing.assert_array_equal(V[:, 1:5], ref[:, 1:5])
    w.X[5, 2] = np.nan
    from paper_1809_11165_amd import binding
    ctx.bbmm_setup(binding.problem_from_workload(w, inputs.ONTHEFLY))
    assert np.isnan(ctx.bbmm_kernel_mm(inputs.ONTHEFLY, Md).cpu().numpy()).all()


@pytest.mark.parametrize("kernel", [inputs.RBF, inputs.MATERN52])
@pytest.mark.parametrize("d", [1, 4, 5, 8, 11, 16])
def test_digit_entries_are_symmetric(ctx, kernel, d):
    """Columns of K for a set of points: entry (i, j) has the bits of entry (j, i) (one digit word each way; an
    iteration with a matrix that is not symmetric takes more steps)."""
    import torch
    n, c = 6200, 32
    w, prob = _problem(n, d, kernel)
    w.X *= np.float32(0.7)
    rows = np.random.default_rng(d).choice(n, size=512, replace=False)
    ctx.bbmm_setup(prob)
    K = np.empty((512, 512), dtype=np.float32)
    for c0 in range(0, 512, c):
        M = np.zeros((n, c), dtype=np.float32)
        M[rows[c0:c0 + c], np.arange(c)] = 1.0
        K[:, c0:c0 + c] = ctx.bbmm_kernel_mm(inputs.ONTHEFLY, torch.from_numpy(M).cuda()).cpu().numpy()[rows]
    assert len(np.unique(K)) > 1000
    np.testing.assert_array_equal(K, K.T)


@pytest.mark.parametrize("kernel", [inputs.RBF, inputs.MATERN52])
@pytest.mark.parametrize("d", [4, 8, 16])
def test_digit_product_is_no_further_off_than_the_fp64_form(ctx, kernel, d):
    """Norm of the error over 1024 rows and 16 columns, against 64 bits.  Both forms share the rounded coordinates and
    norms; what differs is the rounding of the distance's contraction.  2 % for the scatter of 16 384 values."""
    import torch
    n, c = 8000, 16
    w, prob = _problem(n, d, kernel)
    M = np.random.default_rng(d).standard_normal((n, c)).astype(np.float32)
    rows = np.random.default_rng(9).choice(n, size=1024, replace=False)
    ref = _rows(w, rows, M.astype(np.float64))[0]
    ctx.bbmm_setup(prob)
    err = []
    for v in (1, 0):
        ctx.bbmm_tune("otf_sym", v)
        try:
            V = ctx.bbmm_kernel_mm(inputs.ONTHEFLY, torch.from_numpy(M).cuda()).cpu().numpy().astype(np.float64)
        finally:
            ctx.bbmm_tune("otf_sym", 1)
        err.append(np.linalg.norm(V[rows] - ref) / np.linalg.norm(ref))
    print(d, err)
    assert err[0] <= 1.02 * err[1]


@pytest.mark.parametrize("kernel", [inputs.RBF, inputs.MATERN52])
@pytest.mark.parametrize("d,ell", [(16, 1.5), (16, 2.0), (8, 1.0), (4, 0.8), (4, 0.5)])
def test_digit_entries_carry_no_systematic_error(ctx, kernel, d, ell):
    """Row sums of K against the fp64 form's, which shares the rounded coordinates: the roundings of distances and entries
    differ, but their mean over the rows has to vanish within five standard errors.  (RBF entries are 2^-7 ... 2^-14 for the most
    part at d = 16, l = 1.5, where half a unit per entry would show as 2e-8.)"""
    import torch
    n = N0
    w, _ = _problem(n, d, kernel)
    from paper_1809_11165_amd import binding
    w.X = np.random.default_rng(1).standard_normal((n, d)).astype(np.float32)
    w.lengthscale, w.outputscale = np.array([ell]), 1.0
    ctx.bbmm_setup(binding.problem_from_workload(w, inputs.ONTHEFLY))
    one = torch.ones(n, 1, device="cuda")
    V = []
    for v in (1, 0):
        ctx.bbmm_tune("otf_sym", v)
        try:
            V.append(ctx.bbmm_kernel_mm(inputs.ONTHEFLY, one).cpu().numpy().astype(np.float64)[:, 0])
        finally:
            ctx.bbmm_tune("otf_sym", 1)
    e = (V[0] - V[1]) / V[1]
    assert abs(e.mean()) <= 5.0 * e.std() / np.sqrt(n), (e.mean(), e.std() / np.sqrt(n))


@pytest.mark.parametrize("kernel", [inputs.RBF, inputs.MATERN52])
@pytest.mark.parametrize("far", [1e6, 1e13, 1e16, 1e18])
def test_digit_entries_of_a_far_point(ctx, kernel, far):
    """One point very far out (its square still in fp32's range): entries with it are zero, as in the fp64 form.  X is
    centred, so two points on opposite sides keep the others where they are."""
    import torch
    n, d = 6200, 3
    w, _ = _problem(n, d, kernel)
    w.X[17], w.X[4000] = far, -far
    from paper_1809_11165_amd import binding
    ctx.bbmm_setup(binding.problem_from_workload(w, inputs.ONTHEFLY))
    M = torch.from_numpy(np.random.default_rng(2).standard_normal((n, 5)).astype(np.float32)).cuda()
    V = []
    for v in (1, 0):
        ctx.bbmm_tune("otf_sym", v)
        try:
            V.append(ctx.bbmm_kernel_mm(inputs.ONTHEFLY, M).cpu().numpy())
        finally:
            ctx.bbmm_tune("otf_sym", 1)
    assert np.isfinite(V[1]).all()
    np.testing.assert_allclose(V[0][[17, 4000]], (w.outputscale + w.noise) * M.cpu().numpy()[[17, 4000]], rtol=2e-7)
    np.testing.assert_allclose(V[0], V[1], rtol=0, atol=4e-6 * np.abs(V[1]).max())


def _blocks(n):
    """Name, column, whether it suits the digits."""
    rng = np.random.default_rng(n)
    g = rng.standard_normal(n).astype(np.float32)
    one = np.zeros(n, dtype=np.float32)
    one[n // 3] = 1.0
    half = g.copy()
    half[n // 2:] = 0.0
    spike = g.copy()
    spike[5] = 1e12
    few = g.copy()
    few[:n // 16384 + 40] = 0.0
    inf = one.copy()
    inf[n // 3] = np.inf
    nan = g.copy()
    nan[3] = np.nan
    return [("normal", g, True), ("signs", np.sign(g), True), ("zero", 0.0 * one, True), ("uniform", rng.random(n).astype(np.float32), True),
            ("indicator", one, False), ("half zero", half, False), ("one entry far above", spike, False),
            ("lognormal", np.exp(3.0 * g), False), ("a few zeros", few, False), ("infinity", inf, False), ("NaN", nan, False)]


@pytest.mark.parametrize("n,c", [(6200, 5), (6144, 17), (12500, 9), (12500, 17)])
def test_product_takes_the_digits_only_for_blocks_that_suit_them(n, c):
    """By default a block with a column that is not of one size (or a point too far out to be squared) gets the fp64
    product to the bit, and so keeps the accuracy of each row; a dense one gets the digits."""
    import torch
    from paper_1809_11165_amd import binding
    ctx = binding.Context(0)

    def mm(M, **tune):
        for k, v in tune.items():
            ctx.bbmm_tune(k, v)
        try:
            return ctx.bbmm_kernel_mm(inputs.ONTHEFLY, M).cpu().numpy()
        finally:
            for k in tune:
                ctx.bbmm_tune(k, 1)

    w, _ = _problem(n, 6, inputs.RBF)
    w.lengthscale = 0.5 * w.lengthscale
    ctx.bbmm_setup(binding.problem_from_workload(w, inputs.ONTHEFLY))
    fp64 = {"otf_sym": 2 if n >= 12288 and c <= 16 else 0}
    dense = np.random.default_rng(1).standard_normal((n, c)).astype(np.float32)
    for name, col, suits in _blocks(n):
        M = dense.copy()
        M[:, c - 2] = col
        Md = torch.from_numpy(M).cuda()
        V, V64, Vd = mm(Md), mm(Md, **fp64), mm(Md, otf_digits=2)
        np.testing.assert_array_equal(V, Vd if suits else V64, err_msg=name)
        assert not np.array_equal(Vd, V64), name
        if name == "indicator":       # entries of K themselves: seven digits of the smallest as of the largest
            K = O.kernel_block(w.kernel, w.X.astype(np.float64), w.X[n // 3:n // 3 + 1].astype(np.float64), w.lengthscale,
                               w.outputscale)[:, 0]
            small = (K > 1e-12) & (K < 1e-8)
            assert small.sum() > 50 and np.all(np.abs(V[small, c - 2] / K[small] - 1.0) < 1e-4)
    w.X[7], w.X[9] = 1e25, -1e25      # squares overflow: infinitely far from the others
    ctx.bbmm_setup(binding.problem_from_workload(w, inputs.ONTHEFLY))
    Md = torch.from_numpy(dense).cuda()
    V = mm(Md)
    assert np.isfinite(V).all()
    np.testing.assert_array_equal(V, mm(Md, **fp64))
    ctx.close()


@pytest.mark.parametrize("loop_graph", [0, 1])
@pytest.mark.parametrize("kernel", [inputs.RBF, inputs.MATERN52])
def test_calls_with_points_too_far_out_are_those_of_the_fp64_form(kernel, loop_graph):
    """Two points whose squares overflow fp32, on either side of the rest: infinitely far from all others (RBF) or not a
    number (Matern-5/2: infinity times zero).  Whole calls, solves and variances are those of the fp64 form, and
    the next problem has the digits again."""
    import torch
    from paper_1809_11165_amd import binding
    w = inputs.tiny(6300, 3, kernel=kernel, t=4, k=3, iters=12, noise=0.3, seed=4)
    near = w.X.copy()
    far = w.X.copy()
    far[7], far[9] = 1e25, -1e25
    rng = np.random.default_rng(0)
    B = torch.from_numpy(rng.standard_normal((w.n, 6)).astype(np.float32)).cuda()
    Xs = torch.from_numpy(rng.standard_normal((5, 3)).astype(np.float32)).cuda()

    def results(digits, X):
        w.X = X
        ctx = binding.Context(0)
        ctx.bbmm_tune("otf_digits", digits)
        ctx.bbmm_tune("loop_graph", loop_graph)
        out = []
        for _ in range(3):
            ctx.bbmm_setup(binding.problem_from_workload(w, inputs.ONTHEFLY))
            ctx.bbmm_pivoted_cholesky()
            ctx.bbmm_precond_setup()
            U, alpha, beta, resid, iters = ctx.bbmm_mbcg(inputs.ONTHEFLY, B)
            var = ctx.bbmm_predict_var(inputs.ONTHEFLY, Xs)[0]
            out.append([U.cpu().numpy(), alpha, beta, resid, iters, var.cpu().numpy()])
            try:
                r = ctx.bbmm_solve_logdet_grad(binding.problem_from_workload(w, inputs.ONTHEFLY))
                out[-1] += [r.U.cpu().numpy(), r.u0.cpu().numpy(), r.logdet, r.trace, r.quad]
            except RuntimeError as e:
                out[-1].append(str(e))
        ctx.close()
        return out

    for a, b in zip(results(1, far), results(0, far)):
        assert len(a) == len(b)
        if kernel == inputs.RBF:
            assert np.isfinite(a[0]).all() and np.isfinite(a[5]).all()
        for x, y in zip(a, b):
            np.testing.assert_array_equal(x, y)
    a, b = results(1, near)[0], results(0, near)[0]
    assert not np.array_equal(a[1], b[1])
    np.testing.assert_allclose(a[0], b[0], rtol=0, atol=1e-5 * np.abs(b[0]).max())


def test_a_sparse_problem_keeps_no_split_coordinates():
    """Only an exact problem can reach the digit product: 128 bytes per point at d = 8 that an SGPR problem does without."""
    import torch
    from paper_1809_11165_amd import binding
    n = 1 << 19
    w = inputs.tiny_sgpr(n, 8, 16, t=1, k=2, iters=1)
    used = []
    for mode in (inputs.ONTHEFLY, inputs.SGPR):
        ctx = binding.Context(0)
        free = torch.cuda.mem_get_info()[0]
        ctx.bbmm_setup(binding.problem_from_workload(w, mode))
        torch.cuda.synchronize()
        used.append(free - torch.cuda.mem_get_info()[0])
        ctx.close()
    assert used[0] - used[1] >= 120 * n, used


@pytest.mark.parametrize("kernel", [inputs.RBF, inputs.MATERN52])
@pytest.mark.parametrize("c", [3, 18])
@pytest.mark.parametrize("scale", [0, 8, 16, 24, 32, 40])
def test_small_entries_beside_large_ones_that_cancel(ctx, kernel, c, scale):
    """Every weight of the digits counts.  Pairs of equal points carry +1 and -1 times the same value and cancel to the last
    digit; what is left of a row outside them are 600 entries 2^-scale as large, known to the rounding of the entries
    of K as if they stood alone, and to half a unit 2^-62 of the column's largest power of two (4) each.  Without
    the digits of weight 256^-w a row would be off by up to 2^(scale - 8 w) of itself."""
    import torch
    n, d = 6400, 3
    w, _ = _problem(n, d, kernel)
    w.X[1:4000:2] = w.X[0:4000:2]
    from paper_1809_11165_amd import binding
    ctx.bbmm_setup(binding.problem_from_workload(w, inputs.ONTHEFLY))
    rng = np.random.default_rng(scale)
    small = np.zeros((n, c), dtype=np.float32)
    small[4000:4600] = 1.0 + rng.random((600, c), dtype=np.float32)
    small *= np.float32(2.0 ** -scale)
    M = small.copy()
    M[0:4000:2] = (1.0 + rng.random((2000, c))) * np.sign(rng.standard_normal((2000, c)))
    M[1:4000:2] = -M[0:4000:2]
    V = ctx.bbmm_kernel_mm(inputs.ONTHEFLY, torch.from_numpy(M).cuda()).cpu().numpy().astype(np.float64)
    rows = 4600 + rng.choice(n - 4600, size=100, replace=False)
    ref, bound = _rows(w, rows, small.astype(np.float64))
    _check(V[rows], ref, bound + 600 * w.outputscale * 4.0 * 2.0 ** -63)
    assert bound.max() < 1e-4 * np.abs(ref).min()
