"""GPU tests of the projected SGPR iteration, which carries T = A^T D and S = A^T R through their own
recurrences (with A^T A formed once) instead of streaming the root for A^T D in every product.

The streamed iteration is the reference: it is what runs as soon as there is a tolerance to stop at, so
the same problem with a tolerance that no residual meets takes it through the same iterations.  Both work
in fp64 on the same fp32 root.

Two fp64 runs that differ in the order of their sums part ways while a Lanczos process finds eigenvalues
again that it had already found (at sigma^2 = 0.25 the streamed iteration with another number of workgroups
is 4e-5 from itself after 32 iterations, and 0 after 128), so
  * the first eight coefficients are compared at sigma^2 = 0.25: 2^-53 times the condition number (at most |Q| /
    sigma^2 <= n s / sigma^2 = 1.2e5 here) times the length of the sums and the run (a few hundred): 3e-9;
  * solves at sigma^2 = 100, where they converge: they are returned in fp32, 2^-24 of an entry."""
import numpy as np
import pytest

from paper_1809_11165_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

COEFF_TOL = 3e-9
SOLVE_TOL = 6e-8


@pytest.fixture(scope="module")
def ctx():
    from paper_1809_11165_amd import binding
    c = binding.Context(0)
    yield c
    c.close()


def _setup(ctx, n, m, t, k, iters, tol, noise):
    from paper_1809_11165_amd import binding
    w = inputs.make(5, n=n, m=m, t=t, k=k, iters=iters)
    w.noise, w.tol = noise, tol
    prob = binding.problem_from_workload(w, inputs.SGPR)
    prob.pivots_in = np.ascontiguousarray(w.meta["inducing_rows"][:k], dtype=np.int64) if k else None
    return w, prob


def _run(ctx, n, m, k, iters, tol, noise, B):
    _, prob = _setup(ctx, n, m, 1, k, iters, tol, noise)
    ctx.bbmm_setup(prob)
    ctx.bbmm_sgpr_build()
    ctx.bbmm_pivoted_cholesky()
    ctx.bbmm_precond_setup()
    return ctx.bbmm_mbcg(inputs.SGPR, B)


# The smallest n that is projected (2 305 points round up to 2 560 rows, 2 304 = nine 256-row blocks), a ragged one
# and one whose product leaves two partial sums in some rows; one, two, five and eight 128-column
# blocks of A^T A after rounding m to 256; one and two groups of 16 columns; every width of the preconditioner.
@pytest.mark.parametrize("n,m,c,k", [(2304, 1, 1, 0), (2305, 256, 12, 3), (4703, 257, 13, 9), (5003, 1000, 17, 17),
                                     (12289, 130, 16, 16), (30011, 300, 32, 31)])
def test_projected_iteration_is_the_streamed_one(ctx, n, m, c, k):
    iters = max(32, (m + 255) // 256 * 16)
    rng = np.random.default_rng(n)
    B = rng.standard_normal((n, c)).astype(np.float32)
    if c > 2:
        B[:, 1] = 0.0                   # a column that is frozen from the start
        B[n // 2, 2] = np.nan           # one that poisons no other
    B = torch.from_numpy(B).cuda()
    for noise in (0.25, 100.0):
        got = _run(ctx, n, m, k, iters, 0.0, noise, B)
        ref = _run(ctx, n, m, k, iters, 1e-300, noise, B)
        assert got[4] == iters and (ref[4] == iters or m == 1)   # (with m = 1 even 1e-300 is met)
        assert torch.equal(torch.isnan(got[0]), torch.isnan(ref[0]))
        for q in range(c):
            if c > 2 and q in (1, 2):
                continue
            if noise < 1.0:
                # (one inducing point: two eigenvalues, done after two iterations)
                first = 2 if m == 1 else 8
                np.testing.assert_allclose(got[1][:first, q], ref[1][:first, q], rtol=COEFF_TOL, atol=0)
                np.testing.assert_allclose(got[2][:first - 1, q], ref[2][:first - 1, q], rtol=COEFF_TOL, atol=0)
            else:
                u, v = got[0][:, q].double(), ref[0][:, q].double()
                assert float((u - v).norm() / v.norm()) < SOLVE_TOL, q


# wide blocks on more than 256 inducing points are projected from 5 120 (padded) points on only, where that is the faster form
@pytest.mark.parametrize("n,m,c,projected", [(4864, 300, 17, False), (4865, 300, 17, True), (4864, 300, 16, True), (3000, 256, 17, True)])
def test_which_form_runs(ctx, n, m, c, projected):
    B = torch.from_numpy(np.random.default_rng(n).standard_normal((n, c)).astype(np.float32)).cuda()
    got, ref = (_run(ctx, n, m, 3, 32, tol, 0.25, B) for tol in (0.0, 1e-300))
    assert np.array_equal(got[1], ref[1]) != projected


@pytest.mark.parametrize("iters", [32, 50])              # without and with A^T R streamed anew on the way
def test_projected_iteration_repeats_and_alternates(ctx, iters):
    """First pass, recorded and replayed loops give the same bits, also with streamed calls between them."""
    n, m, t, k = 6007, 200, 6, 5
    _, prob = _setup(ctx, n, m, t, k, iters, 0.0, 100.0)
    _, other = _setup(ctx, n, m, t, k, iters, 1e-300, 100.0)
    first = ctx.bbmm_solve_logdet_grad(prob)
    ctx.bbmm_tune("loop_graph", 1)
    try:
        before = ctx.bbmm_loop_graph_stats()
        for _ in range(5):
            mid = ctx.bbmm_solve_logdet_grad(other)
            again = ctx.bbmm_solve_logdet_grad(prob)
            assert torch.equal(first.U, again.U) and first.logdet == again.logdet
            assert np.array_equal(first.alpha, again.alpha)
            assert float((mid.U - first.U).double().norm() / first.U.double().norm()) < SOLVE_TOL
            torch.cuda.synchronize()
        captures, replays = ctx.bbmm_loop_graph_stats()
        assert (captures - before[0], replays - before[1]) == (2, 8)     # of each form the second run is recorded and replayed
    finally:
        ctx.bbmm_tune("loop_graph", 0)


def test_projected_iteration_from_a_warm_start(ctx):
    n, m, t, k, iters = 4099, 64, 4, 5, 32
    _, prob = _setup(ctx, n, m, t, k, iters, 0.0, 100.0)
    _, other = _setup(ctx, n, m, t, k, iters, 1e-300, 100.0)
    u0 = torch.from_numpy(np.random.default_rng(3).standard_normal(n).astype(np.float32)).cuda()
    prob.u0_init = other.u0_init = u0
    a, b = ctx.bbmm_solve_logdet_grad(prob), ctx.bbmm_solve_logdet_grad(other)
    assert float((a.U - b.U).double().norm() / b.U.double().norm()) < SOLVE_TOL


@pytest.mark.parametrize("n,m,c,k", [(20000, 800, 32, 0), (30000, 1024, 16, 10)])
def test_projected_iteration_nears_the_solution_as_the_streamed_one(ctx, n, m, c, k):
    """160 iterations at sigma^2 = 0.25 leave solves some 1e-7 from the 64-bit ones.  Both forms lose iterations to rounding (one
    leaves 0.9 of the distance); the projected one, as a run in 64 bits with plain sums, loses a few more (with A^T R anew every 48
    iterations 1.47 and 1.44 times as far, every 8 1.10 and 1.06, never 1.84 and 1.68): four at most, 0.9^-4 = 1.52."""
    B = torch.from_numpy(np.random.default_rng(n).standard_normal((n, c)).astype(np.float32)).cuda()
    dist = {}
    for tol in (1e-300, 0.0):
        U = _run(ctx, n, m, k, 160, tol, 0.25, B)[0].double()
        A, b = ctx.bbmm_sgpr_root_rows(0, n).double(), B.double()
        At = A.T.contiguous()
        C = At @ A + 0.25 * torch.eye(m, dtype=torch.float64, device="cuda")
        ref = (b - A @ torch.linalg.solve(C, At @ b)) / 0.25
        dist[tol] = float(torch.log((U - ref).norm(dim=0) / ref.norm(dim=0)).mean().exp())
    print(n, m, dist, flush=True)
    assert 3e-8 < dist[1e-300] < 1e-6           # (rounding the solves to fp32 alone: 2.5e-8)
    assert dist[0.0] < 1.52 * dist[1e-300]
