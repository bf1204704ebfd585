"""The multigrid cycle on large levels with a plain shape (more than 1.57M
off-diagonal entries, untiled or by request), where the vectors that tiled and
small levels form in their products' gathers are written first: the same
preconditioner as on the tiled matrix, for every smoother, cycle, prolongation
and depth.  Iteration counts agree to one and solutions to 100 times the
solves' tolerance of the largest entry."""
import numpy as np
import pytest

import synth
from gpu_common import gpu_system, say

pytestmark = pytest.mark.gpu

OPTS = {
    "l1": {},
    "chebyshev1": dict(smoother=1, smoother_degree=1),
    "chebyshev2": dict(smoother=1, smoother_degree=2),
    "chebyshev3": dict(smoother=1, smoother_degree=3),
    "w_smoothed": dict(cycle=2, prolongation=1),
    "k": dict(cycle=3),
}


@pytest.fixture(scope="module")
def ctx():
    from paper_2001_11606_amd import rt
    with rt.Context(0) as c:
        yield c


@pytest.fixture(scope="module")
def problem():
    prob = synth.config3(n=38)   # 54,872 rows; the last tile is ragged
    prob.dt = 0.1
    return prob


@pytest.mark.parametrize("depth", [0, 2, 1])
@pytest.mark.parametrize("name", list(OPTS))
def test_untiled_cycle_is_the_tiled_one(ctx, problem, name, depth):
    import torch
    from paper_2001_11606_amd import rt
    b = torch.tensor(np.random.default_rng(4).uniform(-1.0, 1.0, problem.n_interior),
                     device=ctx.device)
    runs = {}
    for tiled in (1, 0):
        dp, nb, A = gpu_system(ctx, problem, amg=rt.amg_opts(tiled_spmv=tiled, **OPTS[name]))
        info = ctx.matrix_info(A)
        assert info.level_nnz[0] - info.level_n[0] > 3 << 19 and info.levels > 2
        rt.rt_matrix_set_cycle_depth(A, depth)
        for prec, tol in ((0, 1e-12), (1, 1e-11)):
            for shape in ((-1,) if not tiled else (-1, 4)):
                for prod in (0, 1, 2):
                    rt.rt_matrix_set_spmv_shape(A, 0, prod, shape)
                x = torch.zeros_like(b)
                s, st = ctx.solve(A, b, x, rt.solve_opts(prec, 1, tol, 500, 1e-3, 40))
                assert s == rt.RT_OK, rt.rt_last_error()
                runs[tiled, prec, shape] = (st.iterations, x)
        ctx.free(A, nb)
    say(f"[cycle] {name} depth={depth} iterations {[v[0] for v in runs.values()]}")
    for prec, tol in ((0, 1e-12), (1, 1e-11)):
        its, ref = runs[1, prec, -1]
        for key in ((1, prec, 4), (0, prec, -1)):
            assert abs(runs[key][0] - its) <= 1, key
            assert float((runs[key][1] - ref).abs().max()) <= 100 * tol * float(ref.abs().max())
