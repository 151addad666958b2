"""GPU: recorded iteration loops ("loop_graph") beside what changes between the runs that replay them: the problem whose matrix the
loop multiplies by, and the work lists of the size before.  The reference is the same program with every kernel launched."""
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


# every product with a work list laid out for its size: digit words, fp64 triangle, fp64 whole matrix, on the fly by tile pairs, sparse
# streamed and projected
@pytest.mark.parametrize("mode,sym,digits,otf_sym,tol,n1,n2", [
    (inputs.MATERIALISED, 1, 1, 1, 0.0, 8500, 9700), (inputs.MATERIALISED, 1, 0, 1, 0.0, 8500, 9700),
    (inputs.MATERIALISED, 0, 0, 1, 0.0, 8500, 9700), (inputs.ONTHEFLY, 0, 0, 2, 0.0, 3000, 4200),
    (inputs.SGPR, 0, 1, 1, 1e-300, 3000, 4200), (inputs.SGPR, 0, 1, 1, 0.0, 3000, 4200)])
def test_two_sizes_in_turn(mode, sym, digits, otf_sym, tol, n1, n2):
    from paper_1809_11165_amd import binding
    w = {}
    for n in (n1, n2):
        w[n] = inputs.tiny(n, 4, kernel=inputs.RBF, ard=False, t=4, k=5, iters=16, noise=0.5, seed=3)
        if mode == inputs.SGPR:
            w[n] = inputs.with_inducing(w[n], 100, np.random.default_rng(n))
        w[n].tol = tol
    got = {}
    for graph in (0, 1):
        ctx = binding.Context(0)
        for key, value in (("khat_sym", sym), ("otf_digits", digits), ("otf_sym", otf_sym), ("loop_graph", graph)):
            ctx.bbmm_tune(key, value)
        out = []
        for n in [n2] * 4 + [n1] + [n2] * 4 + [n1] * 4 + [n2, n1]:
            out.append(ctx.bbmm_solve_logdet_grad(binding.problem_from_workload(w[n], mode)).U)
            torch.cuda.synchronize()
        assert (ctx.bbmm_loop_graph_stats()[1] > 4) == (graph == 1)
        got[graph] = [a.cpu().numpy() for a in out]
        ctx.close()
    for i, (a, b) in enumerate(zip(got[0], got[1])):
        assert np.array_equal(a, b), i
