"""GPU: recorded iteration loops ("loop_graph") beside what changes between the runs that replay them: the problem whose matrix the
loop multiplies by.  The reference is the same program with every kernel launched."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1809_11165_amd import inputs  # noqa: E402

torch = pytest.importorskip("torch")


# widths that run on the fp32 matrix after a call that has run on digit words alone: 14 columns on the whole matrix and on the triangle,
# 5 columns of a matrix small enough for the product by rows
@pytest.mark.parametrize("n,t,sym,digits,ns", [(11300, 4, 0, 1, 14), (8500, 4, 1, 1, 14), (2100, 19, 0, 2, 5)])
@pytest.mark.parametrize("per_call", [1, 2])
def test_replays_multiply_by_the_matrix_of_the_problem_at_hand(n, t, sym, digits, ns, per_call):
    from paper_1809_11165_amd import binding
    w = inputs.tiny(n, 4, kernel=inputs.RBF, ard=True, t=t, k=5, iters=10, noise=0.5, seed=3)
    Xs = torch.from_numpy(np.ascontiguousarray(w.X[:ns] + np.float32(0.1))).cuda()
    got = {}
    for graph in (0, 1):
        ctx = binding.Context(0)
        for key, value in (("khat_sym", sym), ("otf_digits", digits), ("loop_graph", graph)):
            ctx.bbmm_tune(key, value)
        out = []
        for step in range(6):
            w.noise, w.outputscale = 0.3 + 0.2 * step, 1.0 + 0.5 * step
            out.append(ctx.bbmm_solve_logdet_grad(binding.problem_from_workload(w, inputs.MATERIALISED)).U)
            out += [ctx.bbmm_predict_var(inputs.MATERIALISED, Xs)[0] for _ in range(per_call)]
            torch.cuda.synchronize()
        captures, replays = ctx.bbmm_loop_graph_stats()
        assert (replays > 4) == (graph == 1)
        got[graph] = [a.cpu().numpy() for a in out]
        ctx.close()
    for i, (a, b) in enumerate(zip(got[0], got[1])):
        assert np.array_equal(a, b), i
