"""Kernels of the hierarchy set-up and the cycle at their edges: the blocked dense inverse of
the coarsest level (blocks of 32 rows) at sizes below, at and above multiples
of 32, and the Galerkin product where a coarse row has more distinct columns
than its LDS table takes.  A wrong coarse operator or inverse costs
convergence, so the V-cycle solves must reach the oracle's solution (FP64
1e-12, mixed 1e-10, as in the parity tests) within Jacobi's iterations."""
import numpy as np
import pytest

import synth
from gpu_common import gpu_system, oracle_system, say
from oracle import linsolve

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2001_11606_amd import rt
    with rt.Context(0) as c:
        yield c


def _check(ctx, prob, amg):
    import torch
    from paper_2001_11606_amd import rt
    sysm = oracle_system(prob)[3]
    b = np.random.default_rng(7).standard_normal(prob.n_interior) * sysm.A.diagonal()
    xref = linsolve.dense(sysm.A, b)
    dp, nb, A = gpu_system(ctx, prob, amg=amg)
    info = ctx.matrix_info(A)
    its = {}
    for precond in (0, 1):
        for prec, tol, bar in ((0, 1e-14, 1e-12), (1, 1e-12, 1e-10)):
            bt = torch.tensor(b, device=ctx.device)
            xt = torch.zeros_like(bt)
            status, st = ctx.solve(A, bt, xt, rt.solve_opts(prec, precond, tol, 4000, 1e-4, 60))
            assert status == rt.RT_OK, rt.rt_last_error()
            assert np.max(np.abs(xt.cpu().numpy() - xref)) / np.max(np.abs(xref)) <= bar
            its[(precond, prec)] = st.iterations
    assert its[(1, 0)] <= its[(0, 0)], its
    ctx.free(A, nb)
    return info, its


@pytest.mark.parametrize("n,coarse", [(10, 8), (18, 40), (22, 64), (25, 64), (40, 200), (64, 1024)])
def test_dense_inverse_sizes(ctx, n, coarse):
    from paper_2001_11606_amd import rt
    prob = synth.config1(n=n)
    prob.dt = 0.05
    prob.set_time(prob.dt)
    info, its = _check(ctx, prob, rt.amg_opts(max_levels=8, coarse_size=coarse))
    say(f"[amg set-up] levels {list(info.level_n[:info.levels])} iterations {its}")
    assert info.levels > 1


def test_galerkin_rows_beyond_the_table(ctx):
    from paper_2001_11606_amd import rt
    n = 2200
    rng = np.random.default_rng(23)
    full = lambda v: np.full(n, float(v))   # noqa: E731
    pos = rng.uniform(0.0, 1.0, (3, n))
    prob = synth.Problem(name="crowded", dim=3, pos=pos, h=full(0.3), n_interior=n, m=full(1.0 / n),
                         rho=full(1.0), cv=full(1.0), sigma0_a=full(1.0), sigma_s=full(0.0),
                         opacity_exponent=0.0, e=1.0 + 0.1 * pos[0], E=1.0 + 0.2 * pos[1],
                         Q_e=full(0.0), Q_E=full(0.0), dt=0.1)
    # the higher the threshold, the more particles stay aggregates of their own
    long_rows = 0
    for strength in (0.9, 0.95, 0.98, 0.99, 0.995):
        info, its = _check(ctx, prob, rt.amg_opts(max_levels=2, coarse_size=16, strength=strength))
        row = info.level_nnz[1] / info.level_n[1] if info.levels == 2 else 0.0
        say(f"[amg set-up] strength {strength}: levels {list(info.level_n[:info.levels])}, {row:.0f} "
            f"entries per coarse row, iterations {its}")
        long_rows += row > 400
    assert long_rows, "no hierarchy with coarse rows beyond the table's 384 columns"


@pytest.mark.parametrize("name", ["mms2d_40", "coldpatch3d_12"])
@pytest.mark.parametrize("degree", [0, 1, 2, 3])   # 0: l1-Jacobi, else Chebyshev
def test_cycle_products(ctx, name, degree):
    """The cycle's products with the vector passes in their gathers, on every
    kind of product shape: the small levels' default (plain, restriction in the
    residual's launch), tiled ones (restriction on its own) and a mixture; rows
    outside every aggregate (the cold patch); a coarsest level that is smoothed
    instead of solved (depth 2)."""
    import torch
    from gpu_common import _cold_patch
    from paper_2001_11606_amd import rt
    say(f"[cycle] {name} degree={degree}")
    prob = synth.config1(n=40) if name == "mms2d_40" else _cold_patch(12)
    if name == "mms2d_40":
        prob.dt = 0.05
        prob.set_time(prob.dt)
    sysm = oracle_system(prob)[3]
    b = np.random.default_rng(7).standard_normal(prob.n_interior) * sysm.A.diagonal()
    xref = linsolve.dense(sysm.A, b)
    opts = dict(smoother=rt.RT_SMOOTHER_CHEBYSHEV, smoother_degree=degree) if degree else {}
    dp, nb, A = gpu_system(ctx, prob, amg=rt.amg_opts(max_levels=8, coarse_size=16, **opts))
    levels = ctx.matrix_info(A).levels
    assert levels > 1
    its = {}
    for shapes in ((-1,), (7,), (13,), (4,), (2, 12)):
        for level in range(levels):
            for prec in (0, 1):
                rt.rt_matrix_set_spmv_shape(A, level, prec, shapes[level % len(shapes)])
        for depth in (0, 2):
            rt.rt_matrix_set_cycle_depth(A, depth)
            for prec, tol, bar in ((0, 1e-14, 1e-12), (1, 1e-12, 1e-10)):
                bt = torch.tensor(b, device=ctx.device)
                xt = torch.zeros_like(bt)
                status, st = ctx.solve(A, bt, xt, rt.solve_opts(prec, 1, tol, 4000, 1e-4, 60))
                assert status == rt.RT_OK, rt.rt_last_error()
                assert np.max(np.abs(xt.cpu().numpy() - xref)) / np.max(np.abs(xref)) <= bar
                # the same cycle on every shape: rounding may move a threshold by one
                first = its.setdefault((depth, prec), st.iterations)
                assert abs(st.iterations - first) <= 1 + (prec == 1), (shapes, depth, prec)
    ctx.free(A, nb)
