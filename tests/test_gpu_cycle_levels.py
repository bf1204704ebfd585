"""The V-cycle's way down on either side of its rule: residual and restriction
in one launch up to 4096 aggregates, in two beyond (2-D levels of 70k and 40k
rows over levels of about 10k and 6k, 3-D ones over fewer).  The operator of the
levels is the same either way; each solve against the exported matrix."""
import numpy as np
import pytest
import scipy.sparse as sp

import synth
from gpu_common import gpu_system, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2001_11606_amd import rt
    with rt.Context(0) as c:
        yield c


@pytest.mark.parametrize("opts", [{}, dict(smoother=1, smoother_degree=2), dict(strength=0.0)])
@pytest.mark.parametrize("make", [lambda: synth.config5_member(0, 70000),
                                  lambda: synth.config1(n=200), lambda: synth.config3(n=30)])
def test_levels_above_and_below_the_rule(ctx, make, opts):
    import torch
    from paper_2001_11606_amd import rt
    prob = make()
    dp, nb, A = gpu_system(ctx, prob, amg=rt.amg_opts(**opts))
    info = ctx.matrix_info(A)
    n = prob.n_interior
    rp, col, val, _ = (t.cpu().numpy() for t in ctx.export_matrix(A))
    mat = sp.csr_matrix((val, col, rp), shape=(n, n))
    b = np.random.default_rng(6).uniform(-1.0, 1.0, n) * mat.diagonal()
    its = []
    for prec, tol in ((0, 1e-12), (1, 1e-11)):
        x = torch.zeros(n, dtype=torch.float64, device=ctx.device)
        s, st = ctx.solve(A, torch.tensor(b, device=ctx.device), x,
                          rt.solve_opts(prec, 1, tol, 300, 1e-3, 40))
        assert s == rt.RT_OK, rt.rt_last_error()
        rel = np.linalg.norm(b - mat @ x.cpu().numpy()) / np.linalg.norm(b)
        assert rel <= 1.1 * tol + 1e-14   # the product's order of additions
        its.append(st.iterations)
    say(f"[down] {prob.name} levels {[info.level_n[l] for l in range(info.levels)]} iterations {its}")
    assert max(its) <= 100
    ctx.free(A, nb)
