"""GPU: the finish of the update step by groups of four columns: preconditioner solves over block widths, ranks and
counts of partial rows (whole and partial batches of 32), and the stop over several groups."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1809_11165_amd import inputs  # noqa: E402


@pytest.fixture
def ctx():
    from paper_1809_11165_amd import binding
    c = binding.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n,c,k,blocks", [(1, 1, 0, 0), (40, 4, 1, 0), (900, 5, 8, 0), (8192, 3, 8, 0), (8193, 4, 20, 0),
                                          (20000, 16, 9, 31), (20000, 11, 20, 33), (20000, 17, 20, 128), (20000, 32, 32, 65),
                                          (70000, 13, 5, 512), (70000, 32, 20, 511)])
def test_preconditioner_solve_against_fp64(ctx, n, c, k, blocks):
    """z = (r - L C^-1 L^T r) / s with C = s I + L^T L.  Rounding of a sum over the rows: its longest chain has
    n / 48 + 512 terms of 2^-53; it is carried entry by entry through the solve, once for L^T r and once for C.
    The result is rounded to fp32."""
    import torch
    from paper_1809_11165_amd import binding
    w = inputs.tiny(n, 2, kernel=inputs.MATERN52, t=1, k=k, iters=1, noise=0.5, seed=6)
    ctx.bbmm_tune("ur_blocks", blocks)
    ctx.bbmm_setup(binding.problem_from_workload(w, inputs.ONTHEFLY))
    L = ctx.bbmm_pivoted_cholesky()[0].cpu().numpy()
    ctx.bbmm_precond_setup()
    R = np.random.default_rng(n + c).standard_normal((n, c)).astype(np.float32)
    Z = ctx.bbmm_precond_solve(torch.from_numpy(R).cuda()).cpu().numpy().astype(np.float64)
    R = R.astype(np.float64)
    y = L.T @ R
    Ci = np.linalg.inv(w.noise * np.eye(k) + L.T @ L)
    ref = (R - L @ (Ci @ y)) / w.noise
    aL, aCi = np.abs(L), np.abs(Ci)
    dy = aL.T @ np.abs(R) + (aL.T @ aL) @ (aCi @ np.abs(y))
    bound = 2.0 ** -24 * np.abs(ref) + (n / 48 + 512) * 2.0 ** -53 * (np.abs(R) + aL @ (aCi @ dy)) / w.noise
    assert bound.max() < 1e-4
    assert np.all(np.abs(Z - ref) <= bound), float((np.abs(Z - ref) / bound).max())


@pytest.mark.parametrize("c", [1, 4, 5, 16, 17, 32])
def test_stop_waits_for_every_group(ctx, c):
    import torch
    from paper_1809_11165_amd import binding
    w = inputs.tiny(300, 2, kernel=inputs.RBF, t=1, k=4, iters=64, noise=0.5, seed=2)
    w.tol = 1e-3
    ctx.bbmm_setup(binding.problem_from_workload(w, inputs.MATERIALISED))
    ctx.bbmm_build_khat()
    ctx.bbmm_pivoted_cholesky()
    ctx.bbmm_precond_setup()
    B = torch.from_numpy(np.random.default_rng(c).standard_normal((300, c)).astype(np.float32)).cuda()
    for _ in range(2):
        resid, iters = ctx.bbmm_mbcg(inputs.MATERIALISED, B)[3:]
        assert 0 < iters < 64
        below = (resid[:iters] < w.tol).all(axis=1)
        assert below[-1] and not below[:-1].any()
