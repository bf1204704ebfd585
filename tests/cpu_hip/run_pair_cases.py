"""Drive the pair form of the fine level (matrices without a hierarchy)
through the CPU (AddressSanitizer) build of the library: structure, values,
products, solves, steps and the CSR rows made on demand, against the oracle.
Run like run_cases.py, in a fresh process with libasan preloaded."""
import os
import sys

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path[:0] = [HERE, os.path.dirname(HERE)]
sys.path.insert(0, os.path.dirname(os.path.dirname(HERE)))
os.environ.setdefault("RT_CPU_QUICK", "1")

import synth  # noqa: E402
from gpu_common import _limited, _periodic_x_ghosts_y, _wendland  # noqa: E402
from oracle import linsolve, step as ostep  # noqa: E402
from paper_2001_11606_amd import rt  # noqa: E402
from run_cases import Case, oracle_system, p, rowwise_rel_err, say  # noqa: E402

CASES = {
    # one tile, ragged last tiles, ghosts, two kernels, periodic axes, tiles
    # whose rows have no neighbours right of the diagonal, one particle
    "mms2d_9": lambda: synth.config1(n=9),
    "mms2d_23": lambda: synth.config1(n=23),
    "marshak3d_9": lambda: synth.config4(n=9),
    "density3d_8": lambda: _limited(synth.config3(n=8), synth.LIMITER_LARSEN),
    "wendland3d_8": lambda: _wendland(3, 8),
    "wendland2d_19": lambda: _wendland(2, 19),
    "periodic_x_ghosts_y_18": lambda: _periodic_x_ghosts_y(18),
    "periodic2d_17": lambda: synth.periodic_wendland(2, 17),
    "infinite3d_1": lambda: synth.config2_infinite(1.0, 0.01, n=1),
}


def check(ctx, name, prob):
    ptr, idx, fz, sysm = oracle_system(prob)
    nin = prob.n_interior
    rng = np.random.default_rng(5)
    b = rng.standard_normal(nin) * sysm.A.diagonal()
    xref = linsolve.dense(sysm.A, b)
    c = Case(ctx, prob, amg=rt.amg_opts(max_levels=1))

    def solves(what):
        for prec, tol, bar in ((0, 1e-14, 1e-12), (1, 1e-12, 1e-10)):
            x = np.zeros(nin)
            s, st = rt.rt_solve(ctx, c.A, p(b), p(x), rt.solve_opts(prec, 0, tol, 4000, 1e-4, 60))
            e = np.max(np.abs(x - xref)) / np.max(np.abs(xref))
            assert s == 0 and e <= bar, f"{name}: {what} prec={prec} err={e}"

    solves("pair form")
    info = rt.rt_matrix_get_info(c.A)
    rows = np.repeat(np.arange(nin), np.diff(sysm.A.indptr))
    assert info.nnz == sysm.A.nnz and rows.size == info.nnz
    x = np.zeros(nin)
    s, st = rt.rt_solve_gmres(ctx, c.A, p(b), p(x), rt.gmres_opts(0, 1e-13, 3000, 20))
    assert s == 0 and np.max(np.abs(x - xref)) / np.max(np.abs(xref)) <= 1e-10, f"{name}: gmres"
    ref = ostep.time_step(prob.copy(), fixed_outer=2, solve_tol=1e-15)
    for again in range(2):   # the first assembly, then one on the kept structure
        if again:
            c.A = c.assemble(rt.amg_opts(max_levels=1), c.A)
        e_, E_ = c.arr["e"][:nin].copy(), c.arr["E"][:nin].copy()
        for ell in range(2):
            s, _ = rt.rt_newton_step(ctx, c.A, p(e_), p(E_), ell,
                                     rt.newton_opts(rt.solve_opts(0, 0, 1e-14, 4000)))
            assert s == 0
        assert np.max(np.abs(e_ - ref.e) / ref.e) <= 1e-12, f"{name}: e, assembly {again}"
        assert np.max(np.abs(E_ - ref.E) / ref.E) <= 1e-12, f"{name}: E, assembly {again}"
    # groups in flight (tiled shapes), then CSR rows on demand (a plain shape), then back
    for shape in (8, 13, 16, 0, -1):
        for prec in (0, 1, 2):
            rt.rt_matrix_set_spmv_shape(c.A, 0, prec, shape)
        solves(f"shape {shape}")
    rp, col, val, g, info = c.matrix()
    assert np.array_equal(rp, sysm.A.indptr) and np.array_equal(col, sysm.A.indices), f"{name}: CSR"
    err = rowwise_rel_err(rp, val, sysm.A.data)
    assert err <= 1e-13, f"{name}: values {err}"
    # re-assembled with a hierarchy, and without one again
    c.A = c.assemble(rt.amg_opts(max_levels=8, coarse_size=8), c.A)
    solves("hierarchy")
    c.A = c.assemble(rt.amg_opts(max_levels=1), c.A)
    solves("one level")
    # the neighbour handle freed before the matrix
    d = Case(ctx, prob, amg=rt.amg_opts(max_levels=1))
    rt.rt_neighbors_free(d.nb)
    rt.rt_matrix_set_spmv_shape(d.A, 0, 0, 0)
    x = np.zeros(nin)
    s, st = rt.rt_solve(ctx, d.A, p(b), p(x), rt.solve_opts(0, 0, 1e-14, 4000))
    assert s == 0 and np.max(np.abs(x - xref)) / np.max(np.abs(xref)) <= 1e-12
    rt.rt_matrix_free(d.A)
    c.free()
    say(f"ok {name}: n={nin} nnz={info.nnz} tile columns={info.level_tile_cols[0]}")


def main():
    rt.load(os.environ["RT_CPU_LIB"])
    ctx = rt.rt_create(0, 0)
    want = os.environ.get("RT_CPU_CASES")
    for name, make in CASES.items():
        if not want or name in want.split(","):
            check(ctx, name, make())
    rt.rt_destroy(ctx)
    say("all cases ok")


if __name__ == "__main__":
    main()
