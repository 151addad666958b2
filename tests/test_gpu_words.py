"""GPU: the materialised product from digit words (at most 12 columns: the triangle, panels of 512 columns, tiles of 16; 17 to 32:
the whole matrix, strips of 256) against fp64 kernel rows, and the iterations that run on it against those on the fp64 matrix pipe."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import bbmm_oracle as O  # noqa: E402
from paper_1809_11165_amd import inputs  # noqa: E402

torch = pytest.importorskip("torch")


@pytest.fixture()
def ctx():
    from paper_1809_11165_amd import binding
    c = binding.Context(0)
    c.bbmm_tune("khat_sym", 1)
    yield c
    c.close()


def _workload(n, d, kernel, **kw):
    return inputs.tiny(n, d, kernel=kernel, ard=d > 1, **dict(dict(t=3, k=2, iters=8, noise=0.1, seed=3), **kw))


def _problem(w):
    from paper_1809_11165_amd import binding
    return binding.problem_from_workload(w, inputs.MATERIALISED)


def _rows(w, rows, M):
    """Rows of K_hat M in fp64 and the bound on their error: the distance is fp64 and rounded to fp32 once (2^-24 of
    itself), the kernel function is good to 2^-22 of the entry, the entry is rounded to the fixed-point grid (at the largest
    2^-24 of itself), and the result to fp32."""
    X = w.X.astype(np.float64)
    K = O.kernel_block(w.kernel, X[rows], X, w.lengthscale, w.outputscale)
    xs = X / w.lengthscale
    r2 = ((xs[rows][:, None, :] - xs[None, :, :]) ** 2).sum(axis=2)

    def k(r2):
        if w.kernel == inputs.RBF:
            return w.outputscale * np.exp(-0.5 * r2)
        a = np.sqrt(5.0 * r2)
        return w.outputscale * (1.0 + a + a * a / 3.0) * np.exp(-a)

    dK = k(r2 * (1 - 2.0 ** -24)) - k(r2 * (1 + 2.0 ** -24)) + (2.0 ** -22 + 2.0 ** -24) * K + 0.5 * w.outputscale / 2055208960.0
    dK[np.arange(len(rows)), rows] = 0.0
    K[np.arange(len(rows)), rows] = w.outputscale + w.noise
    ref = K @ M
    return ref, dK @ np.abs(M) + 2.0 ** -23 * np.abs(ref)


# first size with two panels, panels of 256 and 512 columns at the end, pieces of one step and of several; every column count's group
# of four, and the narrowest and widest
@pytest.mark.parametrize("n,c", [(769, 11), (1024, 1), (1025, 4), (1100, 5), (1280, 8), (1281, 9), (1536, 12), (2300, 11), (5000, 3), (9000, 11)])
@pytest.mark.parametrize("kernel,d", [(inputs.RBF, 3), (inputs.MATERN52, 20)])
def test_words_product_against_fp64_rows(ctx, n, c, kernel, d):
    _check_product(ctx, n, c, kernel, d)


def _check_product(ctx, n, c, kernel, d):
    w = _workload(n, d, kernel)
    ctx.bbmm_setup(_problem(w))
    ctx.bbmm_build_khat()
    M = np.random.default_rng(n + c).standard_normal((n, c)).astype(np.float32)
    Mg = torch.from_numpy(M).cuda()
    V64 = ctx.bbmm_kernel_mm(inputs.MATERIALISED, Mg).cpu().numpy()
    ctx.bbmm_tune("otf_digits", 2)
    V = ctx.bbmm_kernel_mm(inputs.MATERIALISED, Mg).cpu().numpy().astype(np.float64)
    ctx.bbmm_tune("otf_digits", 1)
    rows = np.unique(np.r_[0, 15, 16, 511, 512, 767, n // 2, n - 17, n - 1] % n)
    ref, bound = _rows(w, rows, M.astype(np.float64))
    print(n, c, float(np.max(np.abs(V[rows] - ref) / bound)), flush=True)
    assert np.all(np.abs(V[rows] - ref) <= bound)
    assert not np.array_equal(V, V64)                     # the other route did run
    assert np.linalg.norm(V - V64) < 2e-6 * np.linalg.norm(V64)


# first size, an odd number of strips, chunks of equal and unequal length, an odd number of steps in a chunk; the narrowest and widest
# block of every compiled width
@pytest.mark.parametrize("n,c", [(1025, 17), (3841, 17), (4097, 18), (4400, 19), (5000, 24), (7001, 25), (9000, 32), (12300, 21)])
@pytest.mark.parametrize("kernel,d", [(inputs.RBF, 3), (inputs.MATERN52, 20)])
def test_whole_words_product_against_fp64_rows(ctx, n, c, kernel, d):
    ctx.bbmm_tune("khat_sym", 0)
    _check_product(ctx, n, c, kernel, d)


@pytest.mark.parametrize("n,t,sym", [(1100, 10, 1), (2100, 3, 1), (11300, 7, 0), (8000, 16, 0), (16300, 31, 0)])
def test_iteration_on_words_matches_the_fp64_one(ctx, n, t, sym):
    """Both runs are converged, so they solve systems whose entries differ by their evaluation: at most 2^-19 of themselves (the fp32
    distances of the stored matrix lose up to four units of 2^-24 of |x|^2 + |x'|^2 <= 16 here), which moves the solution by
    that times the condition number, at most 1 + (largest row sum) / noise."""
    ctx.bbmm_tune("khat_sym", sym)
    w = _workload(n, 4, inputs.RBF, t=t, k=5, iters=80, noise=4.0)
    X = w.X.astype(np.float64)
    kappa = 1 + max(O.kernel_block(w.kernel, X[i:i + 500], X, w.lengthscale, w.outputscale).sum(axis=1).max() for i in range(0, n, 500)) / w.noise
    ctx.bbmm_setup(_problem(w))
    ctx.bbmm_build_khat()
    ctx.bbmm_pivoted_cholesky()
    ctx.bbmm_precond_setup()
    B = ctx.bbmm_make_probes()
    out = {}
    for dig in (1, 0, 1):
        ctx.bbmm_tune("otf_digits", dig)
        out[dig] = [a.cpu().numpy().astype(np.float64) if torch.is_tensor(a) else a for a in ctx.bbmm_mbcg(inputs.MATERIALISED, B)]
    U1, U0 = out[1][0], out[0][0]
    rel = float(np.linalg.norm(U1 - U0) / np.linalg.norm(U0))
    print(n, t, rel, 2.0 ** -19 * kappa, flush=True)
    assert 0.0 < rel < 2.0 ** -19 * kappa


@pytest.mark.parametrize("n,c,sym,first", [(1500, 4, 1, 12), (11300, 5, 0, 30), (8200, 17, 0, 30), (16400, 25, 0, 60), (20300, 25, 0, 30)])
def test_a_short_run_on_a_built_matrix_takes_its_entries(ctx, n, c, sym, first):
    """Fewer iterations than a conversion to words is worth: the bits of the run without words."""
    ctx.bbmm_tune("khat_sym", sym)
    B = torch.randn(n, c, generator=torch.Generator().manual_seed(1)).cuda()
    for iters in (first - 1, first):
        w = _workload(n, 3, inputs.RBF, t=3, k=2, iters=iters, noise=0.5)
        out = {}
        for dig in (1, 0):
            ctx.bbmm_tune("otf_digits", dig)
            ctx.bbmm_setup(_problem(w))
            ctx.bbmm_build_khat()
            ctx.bbmm_pivoted_cholesky()
            ctx.bbmm_precond_setup()
            out[dig] = ctx.bbmm_mbcg(inputs.MATERIALISED, B)[0].clone()
        assert torch.equal(out[1], out[0]) == (iters < first)


def test_the_fp32_matrix_is_there_after_a_call_that_did_without(ctx):
    n = 11300
    w = _workload(n, 4, inputs.RBF, t=4, k=5, iters=10, noise=0.5)
    ctx.bbmm_solve_logdet_grad(_problem(w))
    K = ctx.bbmm_khat_block(n - 40, 40, 0, 300).cpu().numpy()
    X = w.X.astype(np.float64)
    ref = O.kernel_block(w.kernel, X[n - 40:], X[:300], w.lengthscale, w.outputscale)
    assert np.max(np.abs(K - ref)) < 1e-5
    M = torch.randn(n, 3, device="cuda")
    V = ctx.bbmm_kernel_mm(inputs.MATERIALISED, M).cpu().numpy().astype(np.float64)
    rows = np.array([0, 777, n - 1])
    Kr = O.kernel_block(w.kernel, X[rows], X, w.lengthscale, w.outputscale)
    Kr[np.arange(3), rows] += w.noise
    ref = Kr @ M.cpu().numpy().astype(np.float64)
    assert np.max(np.abs(V[rows] - ref)) < 1e-4


@pytest.mark.parametrize("n,t,sym", [(11300, 4, 0), (8500, 4, 1)])
def test_a_recorded_product_follows_the_calls_that_run_on_words(n, t, sym):
    """A caller's graph of a product reads the fp32 matrix where it was when the product was recorded: after every later call it has to
    be that call's, also one that runs on the digit words."""
    from paper_1809_11165_amd import binding
    stream = torch.cuda.Stream()
    w = _workload(n, 4, inputs.RBF, t=t, k=5, iters=10, noise=0.5)
    M = torch.randn(n, 5, generator=torch.Generator().manual_seed(1)).cuda()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        ctx = binding.Context(0)
        ctx.bbmm_tune("khat_sym", sym)
        ctx.bbmm_solve_logdet_grad(_problem(w))
        ctx.bbmm_kernel_mm(inputs.MATERIALISED, M)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            V = ctx.bbmm_kernel_mm(inputs.MATERIALISED, M)
        for step in range(3):
            w.noise, w.outputscale = 0.4 + 0.3 * step, 1.5 + 0.5 * step
            ctx.bbmm_solve_logdet_grad(_problem(w))
            graph.replay()
            stream.synchronize()
            got = V.clone()
            assert torch.equal(got, ctx.bbmm_kernel_mm(inputs.MATERIALISED, M)), step
            rows = np.array([0, 777, n - 1])
            K = O.kernel_block(w.kernel, w.X[rows].astype(np.float64), w.X.astype(np.float64), w.lengthscale, w.outputscale)
            K[np.arange(3), rows] += w.noise
            assert np.max(np.abs(got.cpu().numpy()[rows] - K @ M.cpu().numpy().astype(np.float64))) < 2e-4, step
        ctx.close()


@pytest.mark.parametrize("had", [0, 1])
@pytest.mark.parametrize("n,t,sym,dig", [(11300, 4, 0, 1), (1500, 4, 1, 1), (11300, 19, 0, 1), (11300, 19, 0, 2)])
def test_a_product_recorded_right_behind_a_call_on_words_holds_no_build(n, t, sym, dig, had):
    """The call leaves no fp32 matrix (had = 1: memory for one, of an earlier build).  A product that is recorded as the first one has to find it
    built, and its replays must neither build it nor read another call's (nor, with otf_digits = 2, words of another form)."""
    from paper_1809_11165_amd import binding
    stream = torch.cuda.Stream()
    w = _workload(n, 4, inputs.RBF, t=t, k=5, iters=10, noise=0.5)
    M = torch.randn(n, 5, generator=torch.Generator().manual_seed(1)).cuda()
    rows = np.array([0, 777, n - 1])
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        ctx = binding.Context(0)
        ctx.bbmm_tune("khat_sym", sym)
        if sym:
            ctx.bbmm_tune("mat_wgs", 256)                  # (keeps the triangle at this size)
        ctx.bbmm_tune("otf_digits", dig)
        if had:
            ctx.bbmm_setup(_problem(w))
            ctx.bbmm_build_khat()
        w.noise, w.outputscale = 0.7, 2.5
        ctx.bbmm_solve_logdet_grad(_problem(w))
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            V = ctx.bbmm_kernel_mm(inputs.MATERIALISED, M)
        for step in range(4):
            if step % 2:
                w.noise, w.outputscale = 0.4 + 0.3 * step, 1.5 + 0.5 * step
                ctx.bbmm_solve_logdet_grad(_problem(w))
            V.zero_()
            graph.replay()
            stream.synchronize()
            got = V.clone()
            assert dig == 2 or torch.equal(got, ctx.bbmm_kernel_mm(inputs.MATERIALISED, M)), step
            K = O.kernel_block(w.kernel, w.X[rows].astype(np.float64), w.X.astype(np.float64), w.lengthscale, w.outputscale)
            K[np.arange(3), rows] += w.noise
            assert np.max(np.abs(got.cpu().numpy()[rows] - K @ M.cpu().numpy().astype(np.float64))) < 2e-4, step
        ctx.close()


def test_words_of_the_other_form_come_from_the_fp32_matrix(ctx):
    """A call leaves the triangle's words (5 columns, nothing in fp32) or the whole matrix's (20); variances at 20 and at 5 points then need
    the other form, whose entries are those of the fp32 matrix: the same bits as on a matrix built by itself."""
    from paper_1809_11165_amd import binding
    n = 11300
    ctx.bbmm_tune("khat_sym", 0)          # (the fixture's default is the triangle)
    w4, w19 = (_workload(n, 4, inputs.RBF, t=t, k=5, iters=30, noise=0.5) for t in (4, 19))
    Xs = torch.from_numpy(np.ascontiguousarray(w4.X[:20] + np.float32(0.1))).cuda()
    with_own = binding.Context(0)
    for w, ns in ((w4, 20), (w19, 5)):
        ctx.bbmm_solve_logdet_grad(_problem(w))
        got = ctx.bbmm_predict_var(inputs.MATERIALISED, Xs[:ns])[0]
        again = ctx.bbmm_predict_var(inputs.MATERIALISED, Xs[:ns])[0]
        with_own.bbmm_setup(_problem(w))
        with_own.bbmm_build_khat()
        with_own.bbmm_pivoted_cholesky()
        with_own.bbmm_precond_setup()
        ref = with_own.bbmm_predict_var(inputs.MATERIALISED, Xs[:ns])[0]
        assert torch.equal(got, ref) and torch.equal(got, again)
    with_own.close()


def _all_but(left):
    """Device memory taken so that `left` bytes can be allocated, in blocks of 32 MB (nothing is written to it)."""
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    block = 32 << 20
    taken = [torch.empty(max(0, torch.cuda.mem_get_info()[0] - left - (8 << 30)), dtype=torch.uint8, device="cuda")]
    try:
        while True:
            taken.append(torch.empty(block, dtype=torch.uint8, device="cuda"))
    except torch.cuda.OutOfMemoryError:
        pass
    del taken[len(taken) - -(-left // block):]
    torch.cuda.empty_cache()
    return taken


def test_the_same_arithmetic_beside_other_users_of_the_device():
    """Words beside a matrix that the caller has had built: by the sizes alone."""
    from paper_1809_11165_amd import binding
    w = _workload(11300, 4, inputs.RBF, t=4, k=5, iters=30, noise=0.5)
    B = torch.randn(w.n, 5, generator=torch.Generator().manual_seed(1)).cuda()
    out = []
    for busy in (False, True):
        own = binding.Context(0)
        own.bbmm_setup(_problem(w))
        own.bbmm_build_khat()
        own.bbmm_pivoted_cholesky()
        own.bbmm_precond_setup()
        other = _all_but(16 << 30) if busy else None
        out.append(own.bbmm_mbcg(inputs.MATERIALISED, B)[0].clone())
        own.close()
        del other
    torch.cuda.empty_cache()
    assert torch.equal(out[0], out[1])


def test_the_matrix_of_an_earlier_problem_gives_way_to_words(ctx):
    """Its memory is idle, and the words of the next problem fit nowhere else."""
    from paper_1809_11165_amd import binding
    ctx.bbmm_tune("khat_sym", 0)
    big, w = (_workload(n, 4, inputs.RBF, t=4, k=5, iters=12, noise=0.5) for n in (30000, 28000))
    ref = ctx.bbmm_solve_logdet_grad(_problem(w)).U
    own = binding.Context(0)
    own.bbmm_tune("otf_digits", 0)
    own.bbmm_solve_logdet_grad(_problem(big))
    own.bbmm_tune("otf_digits", 1)
    ctx.close()
    prob = _problem(w)
    other = _all_but(128 << 20)
    got = own.bbmm_solve_logdet_grad(prob).U
    del other
    own.close()
    torch.cuda.empty_cache()
    assert torch.equal(got, ref)


def test_a_run_whose_words_leave_no_room_for_its_sums_takes_fp32_entries(ctx):
    """Room for the words (1.6 GB) and not for the partial results of products from them (0.2 GB)."""
    ctx.bbmm_tune("khat_sym", 0)
    w = _workload(28000, 4, inputs.RBF, t=4, k=5, iters=30, noise=0.5)
    B = torch.randn(w.n, 5, generator=torch.Generator().manual_seed(1)).cuda()
    ctx.bbmm_setup(_problem(w))
    ctx.bbmm_build_khat()
    ctx.bbmm_pivoted_cholesky()
    ctx.bbmm_precond_setup()
    ctx.bbmm_tune("otf_digits", 0)
    ref = ctx.bbmm_mbcg(inputs.MATERIALISED, B)[0].clone()
    ctx.bbmm_tune("otf_digits", 1)
    panels = 28160 // 512
    other = _all_but((panels * (panels + 1) // 2) * 512 * 512 * 4 + (100 << 20))
    got = ctx.bbmm_mbcg(inputs.MATERIALISED, B)[0].clone()
    del other
    torch.cuda.empty_cache()
    assert torch.equal(got, ref)


def test_points_too_far_out_take_the_fp64_products(ctx):
    n = 1500
    w = _workload(n, 3, inputs.RBF, t=3, k=3, iters=12, noise=0.5)
    X = w.X.copy()
    X[7] = 1e25                                            # its square overflows fp32
    w.X = X
    ctx.bbmm_tune("khat_sym", 1)
    out = {}
    for dig in (1, 0):
        ctx.bbmm_tune("otf_digits", dig)
        ctx.bbmm_setup(_problem(w))
        ctx.bbmm_build_khat()
        ctx.bbmm_pivoted_cholesky()
        ctx.bbmm_precond_setup()
        B = torch.randn(n, 4, generator=torch.Generator().manual_seed(1)).cuda()
        out[dig] = ctx.bbmm_mbcg(inputs.MATERIALISED, B)[0].cpu().numpy()
    assert np.array_equal(out[1], out[0], equal_nan=True)


@pytest.mark.parametrize("n,sym", [(1500, 1), (11300, 0)])
def test_entries_that_are_no_numbers_are_not_hidden_by_the_words(ctx, n, sym):
    """Two opposite points, each with a square below the largest fp32 number and a squared distance above it: the Matern function of that
    pair is infinity times zero in fp32, and a run on the stored matrix says so.  So must one on words, whether they are evaluated
    from X or converted."""
    from paper_1809_11165_amd import binding
    w = _workload(n, 1, inputs.MATERN52, t=3, k=3, iters=30, noise=0.5)
    X = w.X.copy()
    far = 1.6e19 * float(w.lengthscale[0]) / (np.sqrt(5.0) * np.log2(np.e))
    X[7], X[9] = far, -far
    w.X = X
    ctx.bbmm_tune("khat_sym", sym)
    out = {}
    for dig in (0, 1):
        ctx.bbmm_tune("otf_digits", dig)
        ctx.bbmm_setup(_problem(w))
        ctx.bbmm_build_khat()
        ctx.bbmm_pivoted_cholesky()
        ctx.bbmm_precond_setup()
        B = torch.randn(n, 4, generator=torch.Generator().manual_seed(1)).cuda()
        out[dig] = ctx.bbmm_mbcg(inputs.MATERIALISED, B)[0].cpu().numpy()
        with pytest.raises(binding.BbmmError) as e:
            ctx.bbmm_solve_logdet_grad(_problem(w))
        assert e.value.code == binding.ENONFINITE
    assert np.isnan(out[0]).any()
    assert np.array_equal(out[1], out[0], equal_nan=True)
