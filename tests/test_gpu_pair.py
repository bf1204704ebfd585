"""The pair form of the fine level (matrices assembled without a hierarchy):
solves, GMRES, steps, re-assembly, CSR rows on demand and batches against the
oracle, at the edges of its tiles (256 rows), on both kernels, with ghosts,
periodic axes and rows of very different length; tiles that do not fit it; and
the same bits from run to run (its sums are LDS adds in a fixed order).
Tolerances: FP64 solves 1e-12 and mixed ones 1e-10 of the largest entry, as in
the parity tests."""
import numpy as np
import pytest

import synth
from gpu_common import (_limited, _periodic_x_ghosts_y, _wendland, gpu_system, oracle_system,
                        rowwise_rel_err, say)
from oracle import linsolve, step as ostep

pytestmark = pytest.mark.gpu


def _crowded(n):
    """n particles in a few cells: every row couples to most others, so a tile
    has more distinct columns than the tiled forms take."""
    rng = np.random.default_rng(17)
    prob = synth.config2_infinite(1.0, 0.01, n=2)
    pos = rng.uniform(0.0, 1.0, (3, n))
    full = lambda v: np.full(n, float(v))   # noqa: E731
    return synth.Problem(name="crowded", dim=3, pos=pos, h=full(0.35), n_interior=n - 30,
                         m=full(1.0 / n), rho=full(1.0), cv=full(1.0), sigma0_a=full(10.0),
                         sigma_s=full(0.0), opacity_exponent=-3.0, e=1.0 + 0.1 * pos[0],
                         E=1.0 + 0.2 * pos[1], Q_e=full(0.0), Q_E=full(0.0), dt=1e-3,
                         kernel=prob.kernel)


CASES = {
    "mms2d_16 (one full tile, ghosts)": lambda: synth.config1(n=16),
    "mms2d_33": lambda: synth.config1(n=33),
    "infinite3d_1": lambda: synth.config2_infinite(1.0, 0.01, n=1),
    "density3d_11": lambda: _limited(synth.config3(n=11), synth.LIMITER_LARSEN),
    "marshak3d_13": lambda: synth.config4(n=13),
    "wendland3d_10": lambda: _wendland(3, 10),
    "wendland2d_40": lambda: _wendland(2, 40),
    "periodic3d_13": lambda: synth.periodic_wendland(3, 13),
    "periodic_x_ghosts_y_21": lambda: _periodic_x_ghosts_y(21),
    "crowded_3600 (untiled)": lambda: _crowded(3600),
}


@pytest.fixture(scope="module")
def ctx():
    from paper_2001_11606_amd import rt
    with rt.Context(0) as c:
        yield c


def _solve(ctx, A, b, precision, tol):
    import torch
    from paper_2001_11606_amd import rt
    bt = torch.tensor(b, device=ctx.device)
    xt = torch.zeros_like(bt)
    status, st = ctx.solve(A, bt, xt, rt.solve_opts(precision, 0, tol, 4000, 1e-4, 60))
    assert status == rt.RT_OK, rt.rt_last_error()
    return xt.cpu().numpy()


@pytest.mark.parametrize("name", list(CASES))
def test_pair_form_against_oracle(ctx, name):
    import torch
    from paper_2001_11606_amd import driver, rt
    say(f"[pair] {name}")
    prob = CASES[name]()
    ptr, idx, fz, sysm = oracle_system(prob)
    nin = prob.n_interior
    b = np.random.default_rng(5).standard_normal(nin) * sysm.A.diagonal()
    xref = linsolve.dense(sysm.A, b)
    scale = np.max(np.abs(xref))
    one = rt.amg_opts(max_levels=1)
    dp, nb, A = gpu_system(ctx, prob, amg=one)

    def solves():
        for prec, tol, bar in ((0, 1e-14, 1e-12), (1, 1e-12, 1e-10)):
            x = _solve(ctx, A, b, prec, tol)
            assert np.max(np.abs(x - xref)) / scale <= bar
            assert np.array_equal(x, _solve(ctx, A, b, prec, tol))   # the same bits

    solves()
    bt = torch.tensor(b, device=ctx.device)
    xt = torch.zeros_like(bt)
    status, _ = ctx.solve_gmres(A, bt, xt, rt.gmres_opts(0, 1e-13, 3000, 20))
    assert status == rt.RT_OK and np.max(np.abs(xt.cpu().numpy() - xref)) / scale <= 1e-10
    ref = ostep.time_step(prob.copy(), fixed_outer=2, solve_tol=1e-15)
    for again in (0, A):   # a fresh matrix, then values on the kept structure
        e, E, M, rep = driver.time_step(ctx, dp, nb, A=again, amg=one,
                                        solve=rt.solve_opts(0, 0, 1e-14, 4000), fixed_outer=2)
        assert np.max(np.abs(e.cpu().numpy() - ref.e) / ref.e) <= 1e-12
        assert np.max(np.abs(E.cpu().numpy() - ref.E) / ref.E) <= 1e-12
    # groups in flight (tiled shapes), CSR rows on demand (a plain shape), back
    for shape in (8, 13, 16, 4, -1):
        for prod in (0, 1, 2):
            rt.rt_matrix_set_spmv_shape(A, 0, prod, shape)
        solves()
    rp, col, val, g = (t.cpu().numpy() for t in ctx.export_matrix(A))
    assert np.array_equal(rp, sysm.A.indptr) and np.array_equal(col, sysm.A.indices)
    assert rowwise_rel_err(rp, val, sysm.A.data) <= 1e-13
    # re-assembled with a hierarchy on the same handle, and without one again
    for levels in (8, 1):
        ctx.assemble(nb, dp.arrays, dp.dt, dp.c, dp.a, dp.opacity_exponent, dp.limiter,
                     dp.limiter_k, amg=rt.amg_opts(max_levels=levels, coarse_size=16), A=A)
        solves()


def test_matrix_outlives_neighbour_handle(ctx):
    """The neighbour lists stay with the matrix when their handle is freed
    first: the CSR rows a plain shape asks for are made from them."""
    from paper_2001_11606_amd import rt
    prob = synth.config1(n=20)
    sysm = oracle_system(prob)[3]
    b = np.random.default_rng(6).standard_normal(prob.n_interior) * sysm.A.diagonal()
    xref = linsolve.dense(sysm.A, b)
    dp, nb, A = gpu_system(ctx, prob, amg=rt.amg_opts(max_levels=1))
    ctx.free(nb)
    for shape in (-1, 2):
        rt.rt_matrix_set_spmv_shape(A, 0, rt.RT_PREC_FP64, shape)
        x = _solve(ctx, A, b, 0, 1e-14)
        assert np.max(np.abs(x - xref)) / np.max(np.abs(xref)) <= 1e-12


@pytest.mark.parametrize("n,restart", [(1, 4), (20, 4), (93, 12)])
def test_gmres_sizes(ctx, n, restart):
    """GMRES with one and with four elements per thread in its basis passes
    (804k rows), cut off inside a cycle and run to the end: the residual it
    reports is that of the exported matrix (summation order apart)."""
    import scipy.sparse as sp
    import torch
    from paper_2001_11606_amd import rt
    dp, nb, A = gpu_system(ctx, synth.config3(n=n), amg=rt.amg_opts(max_levels=1))
    nin = dp.n_interior
    rp, col, val, _ = (t.cpu().numpy() for t in ctx.export_matrix(A))
    mat = sp.csr_matrix((val, col, rp), shape=(nin, nin))
    V = (dp.arrays["m"] / dp.arrays["rho"])[:nin].cpu().numpy()
    bt = torch.tensor(np.random.default_rng(8).standard_normal(nin) * V, device=ctx.device)

    def run(max_iter):
        xt = torch.zeros_like(bt)
        status, st = ctx.solve_gmres(A, bt, xt, rt.gmres_opts(0, 1e-11, max_iter, restart))
        b, x = bt.cpu().numpy(), xt.cpu().numpy()
        rel = np.linalg.norm((b - mat @ x) / V) / np.linalg.norm(b / V)
        assert abs(rel - st.rel_residual) <= 1e-6 * rel + 1e-14
        return status, st, x

    status, st, x = run(3000)
    assert status == rt.RT_OK and st.rel_residual <= 1e-11
    assert np.array_equal(x, run(3000)[2])   # the same bits
    for cut in (1, 3, restart + 1):
        if cut < st.iterations:
            s, c, _ = run(cut)
            assert s == rt.RT_NOT_CONVERGED and c.iterations == cut


@pytest.mark.parametrize("mixed_forms", [False, True])
def test_batch_of_pair_form_matrices(ctx, mixed_forms):
    """A batch whose matrices all have the pair form takes it over (also after
    the matrices are freed, and for every requested shape); one matrix with
    CSR rows makes a CSR batch.  Every problem against the oracle."""
    import torch
    from paper_2001_11606_amd import rt
    probs = [synth.config1(n=16), synth.config4(n=9), _wendland(3, 7), synth.config1(n=23)]
    built, refs, bs = [], [], []
    for q, prob in enumerate(probs):
        levels = 8 if mixed_forms and q == 1 else 1
        built.append(gpu_system(ctx, prob, amg=rt.amg_opts(max_levels=levels)))
        sysm = oracle_system(prob)[3]
        bs.append(np.random.default_rng(q).standard_normal(prob.n_interior) * sysm.A.diagonal())
        refs.append(linsolve.dense(sysm.A, bs[-1]))
    B = rt.rt_batch_create(ctx.handle, [A for _, _, A in built])
    ctx.free(*[h for _, nb, A in built for h in (A, nb)])
    b = torch.tensor(np.concatenate(bs), device=ctx.device)
    for prec, tol, bar in ((0, 1e-14, 1e-12), (1, 1e-12, 1e-10)):
        for shape, graph in ((-1, 0), (-1, 3), (16, 0), (3, 2)):
            for prod in (0, 1, 2):
                rt.rt_batch_set_spmv_shape(B, prod, shape)
            x = torch.zeros_like(b)
            s, _ = rt.rt_batch_solve(ctx.handle, B, len(probs), b.data_ptr(), x.data_ptr(),
                                     rt.solve_opts(prec, 0, tol, 4000, 1e-4, 60), graph)
            assert s == rt.RT_OK
            o = 0
            for q, ref in enumerate(refs):
                got = x[o:o + ref.size].cpu().numpy()
                o += ref.size
                assert np.max(np.abs(got - ref)) / np.max(np.abs(ref)) <= bar, (q, prec, shape)
    rt.rt_batch_free(B)


@pytest.mark.parametrize("n,shape", [(82, -1), (82, 4), (33, 4), (20, -1)])
@pytest.mark.parametrize("precond", [0, 1])
def test_batch_reductions(ctx, n, shape, precond):
    """Problems with more partials than the batch's update kernels sum
    themselves (2048 tiles; a plain shape has 16 rows per partial), beside a
    small one that stops first and a zero right-hand side (stops at once).  Every
    problem against its own solve: x to the sum of both solves' bars."""
    import torch
    from paper_2001_11606_amd import rt
    say(f"[batch sums] n={n} shape={shape} precond={precond}")
    levels = 8 if precond else 1
    probs = [synth.config3(n=n), synth.config4(n=9), synth.config3(n=12)]
    built = [gpu_system(ctx, p, amg=rt.amg_opts(max_levels=levels, build_fp32=1)) for p in probs]
    mats = [A for _, _, A in built]
    rng = np.random.default_rng(11)
    bs = [torch.tensor(rng.standard_normal(p.n_interior), device=ctx.device) for p in probs]
    bs[2].zero_()
    B = rt.rt_batch_create(ctx.handle, mats)
    b = torch.cat(bs)
    for prec, tol, bar in ((0, 1e-13, 1e-11), (1, 1e-11, 1e-9)):
        opts = rt.solve_opts(prec, precond, tol, 4000, 1e-4, 60)
        refs = []
        for A, bp in zip(mats, bs):
            x = torch.zeros_like(bp)
            assert ctx.solve(A, bp, x, opts)[0] == rt.RT_OK
            refs.append(x)
        for prod in (0, 1, 2):
            rt.rt_batch_set_spmv_shape(B, prod, shape)
        runs = []
        for graph in (0, 3, 0):
            x = torch.zeros_like(b)
            s, stats = rt.rt_batch_solve(ctx.handle, B, len(probs), b.data_ptr(), x.data_ptr(),
                                         opts, graph)
            assert s == rt.RT_OK
            for got, ref in zip(x.split([r.numel() for r in refs]), refs):
                scale = max(float(ref.abs().max()), 1e-300)
                assert float((got - ref).abs().max()) <= 2 * bar * scale
            runs.append(x)
        assert torch.equal(runs[0], runs[2])   # the same bits
        assert stats[2].iterations == 0 and stats[0].iterations > 0
    rt.rt_batch_free(B)
    ctx.free(*[h for _, nb, A in built for h in (A, nb)])
