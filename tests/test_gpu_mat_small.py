"""GPU: the materialised product by 64-column workgroups (16-column blocks, up to 8192 padded rows) at the edges of
its row chunks, of the block widths and of the sizes that it takes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1809_11165_amd import inputs  # noqa: E402


@pytest.mark.parametrize("n,c", [(1, 1), (16, 12), (255, 16), (256, 11), (257, 13), (1000, 11), (1000, 16), (2500, 12),
                                 (2561, 1), (5000, 13), (8192, 11), (8192, 16), (8193, 11), (8193, 16)])
def test_small_materialised_product_against_stored_rows(n, c):
    """Products and sums in fp64 over the stored fp32 entries: n roundings of 2^-53 of the sum of magnitudes, and the
    final rounding of the result to fp32."""
    import torch
    from paper_1809_11165_amd import binding
    w = inputs.tiny(n, 3, kernel=inputs.RBF, ard=True, t=1, k=1, iters=1, noise=0.1, seed=5)
    ctx = binding.Context(0)
    try:
        ctx.bbmm_setup(binding.problem_from_workload(w, inputs.MATERIALISED))
        ctx.bbmm_build_khat()
        M = np.random.default_rng(n + c).standard_normal((n, c)).astype(np.float32)
        V = ctx.bbmm_kernel_mm(inputs.MATERIALISED, torch.from_numpy(M).cuda()).cpu().numpy().astype(np.float64)
        K = ctx.bbmm_khat_block(0, n, 0, n).cpu().numpy().astype(np.float64)
    finally:
        ctx.close()
    M = M.astype(np.float64)
    ref = K @ M
    bound = 2.0 ** -24 * np.abs(ref) + 2 * (n + 2) * 2.0 ** -53 * (np.abs(K) @ np.abs(M))
    assert np.all(np.abs(V - ref) <= bound), float((np.abs(V - ref) / bound).max())
