"""GPU: long sums of the ARD derivative terms (row blocks summed in fp32 for 32 blocks at a time, fp64 beyond)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1809_11165_amd import inputs  # noqa: E402


def _quad64(w, u):
    """u^T (dK/dl_d) u for every dimension in 64 bits (Matern-5/2)."""
    import torch
    ls = torch.from_numpy(np.broadcast_to(w.lengthscale, (w.d,)).copy()).cuda()
    X = torch.from_numpy(w.X).cuda().double() / ls
    u = u.double()
    out = torch.zeros(w.d, dtype=torch.float64, device="cuda")
    sq = (X * X).sum(1)
    for i in range(0, w.n, 4000):
        xi, ui = X[i:i + 4000], u[i:i + 4000]
        rho = (sq[i:i + 4000, None] + sq[None, :] - 2.0 * (xi @ X.T.contiguous())).clamp_(min=0.0).sqrt_().mul_(5.0 ** 0.5)
        T = (1.0 + rho).mul_(torch.exp(-rho)).mul_(w.outputscale * 5.0 / 3.0)
        T.mul_(ui[:, None]).mul_(u[None, :])
        out += 2.0 * (xi * xi * T.sum(1)[:, None]).sum(0) - 2.0 * (xi * (T @ X)).sum(0)
    return (out / ls).cpu().numpy()


@pytest.mark.parametrize("seed", [4, 7])
def test_long_sums_do_not_lose_to_their_length(seed):
    """Quad terms of positive weights, n = 50 000, d = 16: nothing cancels, so the entries' own rounding leaves at most 2^-23.
    fp32 sums over runs of 32 row blocks (512 terms a lane) add a random walk of sqrt(512) 2^-25 per run, which the
    thousands of runs average out; a quarter of 2^-23 is allowed for it.  (Over a whole chunk of 150 blocks the
    small terms that follow are rounded against the full sum alike in all chunks: 2e-7 and 3e-7 here.)"""
    import torch
    from paper_1809_11165_amd import binding
    w = inputs.make(3, n=50000, t=10, k=0, iters=1, salt=1 + seed)
    assert w.kernel == inputs.MATERN52 and w.d == 16 and len(w.lengthscale) == 16
    rng = np.random.default_rng(seed)
    U = torch.from_numpy(np.abs(rng.standard_normal((w.n, 11), dtype=np.float32))).cuda()
    W = torch.from_numpy(rng.standard_normal((w.n, 10), dtype=np.float32)).cuda()
    ctx = binding.Context(0)
    ctx.bbmm_setup(binding.problem_from_workload(w, inputs.ONTHEFLY))
    quad = np.asarray(ctx.bbmm_dk_traces(U, W)[1])[:16]
    ctx.close()
    ref = _quad64(w, U[:, 0])
    assert np.linalg.norm(quad - ref) <= 1.25 * 2.0 ** -23 * np.linalg.norm(ref), np.linalg.norm(quad - ref) / np.linalg.norm(ref)
