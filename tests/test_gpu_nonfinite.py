"""An initial guess or state with an infinite entry: the residual b - A x is
infinite (a row's sum takes in its own columns only, no zero entry that only
fills up a load or a group meets it), so solves report RT_NOT_CONVERGED with
an infinite relative residual and leave x as it was, GMRES fails with
RT_E_DEVICE, and the backward-Euler residual is infinite."""
import numpy as np
import pytest

import synth
from gpu_common import _wendland, gpu_system

pytestmark = pytest.mark.gpu

CASES = {
    "mms2d_21": lambda: synth.config1(n=21),
    "density3d_9": lambda: synth.config3(n=9),
    "wendland3d_8": lambda: _wendland(3, 8),
}


@pytest.fixture(scope="module")
def ctx():
    from paper_2001_11606_amd import rt
    with rt.Context(0) as c:
        yield c


def _check(ctx, prob, amg, shapes=(-1,)):
    import torch
    from paper_2001_11606_amd import rt
    dp, nb, A = gpu_system(ctx, prob, amg=amg)
    n = prob.n_interior
    b = torch.tensor(np.random.default_rng(2).uniform(0.5, 1.0, n), device=ctx.device)
    for shape in shapes:
        for prod in (0, 1, 2):
            rt.rt_matrix_set_spmv_shape(A, 0, prod, shape)
        for at in (0, n // 2, n - 1):   # rows with and without pairs right of the diagonal
            x0 = torch.ones_like(b)
            x0[at] = float("inf")
            for prec in (0, 1):
                x = x0.clone()
                s, st = ctx.solve(A, b, x, rt.solve_opts(prec, 0, 1e-10, 200))
                assert s == rt.RT_NOT_CONVERGED and st.iterations == 0, (shape, at, prec)
                assert st.rel_residual == np.inf and st.init_rel_residual == np.inf
                assert torch.equal(x, x0)
            with pytest.raises(rt.RtError) as ei:
                ctx.solve_gmres(A, b, x0.clone(), rt.gmres_opts(0, 1e-10, 100, 10))
            assert ei.value.code == rt.RT_E_DEVICE
            e = dp.arrays["e"][:n].clone()
            assert ctx.newton_residual(A, e, x0).rad_norm == np.inf
    ctx.free(A, nb.handle)


@pytest.mark.parametrize("name", list(CASES))
def test_pair_form_infinite_entry(ctx, name):
    from paper_2001_11606_amd import rt
    _check(ctx, CASES[name](), rt.amg_opts(max_levels=1))


@pytest.mark.parametrize("name", list(CASES))
def test_csr_rows_infinite_entry(ctx, name):
    """A matrix with a hierarchy (its small fine level takes a plain shape by
    default), then every kind of requested shape."""
    from paper_2001_11606_amd import rt
    _check(ctx, CASES[name](), rt.amg_opts(max_levels=8, coarse_size=16),
           shapes=(-1, 0, 1, 2, 3, 4, 5, 6, 8, 13, 16))


@pytest.mark.parametrize("levels", [1, 8])
def test_guess_that_is_not_a_number(ctx, levels):
    """No iterations and no refinements on a residual that is not a number."""
    import torch
    from paper_2001_11606_amd import rt
    prob = synth.config1(n=21)
    dp, nb, A = gpu_system(ctx, prob, amg=rt.amg_opts(max_levels=levels, coarse_size=16))
    b = torch.ones(prob.n_interior, dtype=torch.float64, device=ctx.device)
    for prec in (0, 1):
        x = torch.ones_like(b)
        x[7] = float("nan")
        _, st = ctx.solve(A, b, x, rt.solve_opts(prec, 0, 1e-10, 200))
        assert st.iterations == 0 and st.refinements == 0 and np.isnan(st.rel_residual), prec
        assert torch.isnan(x[7]) and int((x == 1.0).sum()) == prob.n_interior - 1
    ctx.free(A, nb)
