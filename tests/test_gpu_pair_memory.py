"""Device memory of matrices whose tiles do not fit the pair form: CSR rows and
the 16-bit columns of the tiled form, nothing of the pair form."""
import pytest

from gpu_common import gpu_system, say
from test_gpu_pair import _crowded

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2001_11606_amd import rt
    with rt.Context(0) as c:
        yield c


def _held(ctx, amg):
    """Bytes held by a matrix of the crowded problem, and its entries."""
    import torch
    from paper_2001_11606_amd import rt
    dp, nb, A = gpu_system(ctx, _crowded(3600), amg=rt.amg_opts(max_levels=1, build_fp32=0))
    ctx.free(A)
    rt.rt_release_cached(ctx.handle)
    free = torch.cuda.mem_get_info()[0]
    A = ctx.assemble(nb, dp.arrays, dp.dt, dp.c, dp.a, dp.opacity_exponent, dp.limiter,
                     dp.limiter_k, amg=amg)
    torch.cuda.synchronize()
    rt.rt_release_cached(ctx.handle)
    held = free - torch.cuda.mem_get_info()[0]
    nnz = ctx.matrix_info(A).nnz
    ctx.free(A, nb)
    return held, nnz


def test_untiled_matrix_holds_no_pair_form(ctx):
    from paper_2001_11606_amd import rt
    plain, nnz = _held(ctx, rt.amg_opts(max_levels=1, build_fp32=0, tiled_spmv=0))
    tried, _ = _held(ctx, rt.amg_opts(max_levels=1, build_fp32=0, tiled_spmv=1))
    say(f"[memory] nnz={nnz} plain {plain} tried {tried}")
    assert nnz > 4_000_000   # the pair form's columns take 2 bytes an entry as well
    assert tried - plain <= 2 * nnz + (6 << 20)   # the tiled form's columns, and rounding


@pytest.mark.parametrize("batch", [False, True])
def test_tuning_keeps_rows_only_for_a_plain_choice(ctx, batch):
    """rt_matrix_tune and rt_batch_tune make CSR rows to time the plain shapes
    (16 bytes an entry with FP32); 64^3 particles choose the pair form, and the
    rows are given back."""
    import torch
    import synth
    from paper_2001_11606_amd import rt
    dp, nb, A = gpu_system(ctx, synth.config3(n=64), amg=rt.amg_opts(max_levels=1))
    B = rt.rt_batch_create(ctx.handle, [A]) if batch else None
    nnz = ctx.matrix_info(A).nnz
    torch.cuda.synchronize()
    rt.rt_release_cached(ctx.handle)
    free = torch.cuda.mem_get_info()[0]
    if batch:
        rep = rt.rt_batch_tune(ctx.handle, B, 3)
        chosen = [rep.chosen[0][p] for p in range(3)]
    else:
        chosen = ctx.tune(A, 3)["chosen"][0]
    torch.cuda.synchronize()
    rt.rt_release_cached(ctx.handle)
    held = free - torch.cuda.mem_get_info()[0]
    say(f"[memory] chosen {chosen}, held after the tuner {held}")
    shapes = rt.rt_spmv_shapes()
    plain = [c for c in chosen if c >= 0 and not shapes[c][2]]
    assert held >= 12 * nnz if plain else held <= 4 << 20
    if B:
        rt.rt_batch_free(B)
    ctx.free(A, nb)


def test_tiles_follow_the_columns(ctx):
    """Across the row lengths at which tiles stop to fit, a matrix without a
    hierarchy (pair form, else tiles, else neither) reports the tile columns of
    the CSR build of one with a hierarchy."""
    import numpy as np
    import torch
    import synth
    from gpu_common import _wendland
    from paper_2001_11606_amd import rt
    seen = set()
    for support in (3.0, 4.0, 4.6, 4.8, 5.0, 5.2, 5.4, 6.0):
        prob = _wendland(3, 18)
        prob.h = np.full_like(prob.h, support / 18)
        dp, nb, A = gpu_system(ctx, prob, amg=rt.amg_opts(max_levels=1))
        H = ctx.assemble(nb, dp.arrays, dp.dt, dp.c, dp.a, dp.opacity_exponent, dp.limiter,
                         dp.limiter_k, amg=rt.amg_opts(max_levels=8))
        a, h = ctx.matrix_info(A), ctx.matrix_info(H)
        say(f"[tiles] support {support}: {a.nnz / a.n:.0f} entries a row, "
            f"{a.level_tile_cols[0]} tile columns")
        assert a.nnz == h.nnz and a.level_tile_cols[0] == h.level_tile_cols[0]
        seen.add(a.level_tile_cols[0] > 0)
        b = torch.ones(prob.n_interior, dtype=torch.float64, device=ctx.device)
        xs = []
        for M in (A, H):
            x = torch.zeros_like(b)
            s, _ = ctx.solve(M, b, x, rt.solve_opts(0, 0, 1e-12, 2000))
            assert s == rt.RT_OK
            xs.append(x)
        assert float((xs[0] - xs[1]).abs().max()) <= 1e-10 * float(xs[1].abs().max())
        ctx.free(A, H, nb)
    assert seen == {False, True}
