"""Many right-hand sides on the tiles of 16 rows (matrix-core products):
widths at the edges of their padding (16, multiples of 32), level sizes that
are no multiple of a tile or of a 64-row block, coarser levels more than 65536
columns away, FP64, FP32 with FP64 values, and FP32 with remainders.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _run(sizes, R, mode, pick):
    """Columns `pick` of one solve with R right-hand sides against the
    single-right-hand-side solves of the same columns; every column's residual."""
    import paper_2503_04914_amd as m

    h = synth.halton_hierarchy(sizes=sizes)
    F = np.ascontiguousarray(np.stack([synth.fourier_target(3900 + r)(h.points) for r in range(R)], axis=1))
    ctx = m.mskm_create(0)
    hd = m.mskm_hier_create(ctx, h.points, h.offsets, h.delta, fp64=mode != "split", fp32=mode != "fp64")
    kw = dict(algorithm=m.MSKM_ALG_SEQUENTIAL, precond=m.MSKM_PRECOND_BLOCK_JACOBI)
    o = m.solve_opts(cg_rtol=1e-13, **kw) if mode == "fp64" else \
        m.solve_opts(precision=m.MSKM_PREC_FP32, cg_rtol=1e-5, target_rel_residual=1e-13, max_refine=20, **kw)
    try:
        A = np.zeros_like(F)
        r = m.mskm_solve(ctx, hd, F, A, o, nrhs=R)
        assert r.status == m.MSKM_OK, r.report
        # FP64 arithmetic on residuals of 1e-13: an order of magnitude of room for their own rounding
        assert m.mskm_residual(ctx, hd, A, F, nrhs=R).max() <= 1e-12
        for c in pick:
            a = np.zeros(len(F))
            assert m.mskm_solve(ctx, hd, np.ascontiguousarray(F[:, c]), a, o).status == m.MSKM_OK
            # both within the repository's bars (1e-10 FP64, 1e-8 mixed) of the exact coefficients
            bar = 2e-10 if mode == "fp64" else 2e-8
            for l in range(h.levels):
                sl = slice(h.offsets[l], h.offsets[l + 1])
                assert np.linalg.norm(A[sl, c] - a[sl]) <= bar * np.linalg.norm(a[sl]), (c, l)
    finally:
        m.mskm_hier_destroy(hd)
        m.mskm_destroy(ctx)


@pytest.mark.parametrize("mode", ["fp64", "fp32", "split"])
@pytest.mark.parametrize("R", [2, 16, 17, 33, 96, 320])
def test_widths(R, mode):
    _run([15, 81, 1030], R, mode, sorted({0, R // 2, R - 1}))


def test_far_columns():
    """Lower rows whose columns lie in windows more than 65536 columns apart (FP64: the third level is
    nearly solved by the second, so a per-level bar on its small coefficients needs the tight solve)."""
    _run([40, 70001, 70003], 3, "fp64", [1])


@pytest.mark.parametrize("nrhs", [1, 2, 15, 16, 530])
def test_residuals_at_once(nrhs):
    """Residuals of several right-hand sides at once against one by one (the
    same FP64 products in another order: 1e-12 of residuals of order one), before
    and after a solve has built the tiles; a batch reports per group."""
    import paper_2503_04914_amd as m

    hs = [synth.halton_hierarchy(sizes=[9, 70, 515]), synth.halton_hierarchy(sizes=[33, 130], start=7001)]
    N = sum(h.n_total for h in hs)
    rng = np.random.default_rng(11)
    A, F = rng.standard_normal((N, nrhs)), rng.standard_normal((N, nrhs))
    ctx = m.mskm_create(0)
    hd = m.mskm_hier_create_batch(ctx, [(h.points, h.offsets, h.delta) for h in hs])
    try:
        one = np.concatenate([m.mskm_residual(ctx, hd, np.ascontiguousarray(A[:, r]), np.ascontiguousarray(F[:, r]))
                              for r in range(nrhs)])
        np.testing.assert_allclose(m.mskm_residual(ctx, hd, A, F, nrhs=nrhs), one, rtol=1e-12)
        X = np.zeros((N, 3))
        m.mskm_solve(ctx, hd, np.ascontiguousarray(np.ones((N, 3))), X, m.solve_opts(cg_rtol=1e-6), nrhs=3)
        np.testing.assert_allclose(m.mskm_residual(ctx, hd, A, F, nrhs=nrhs), one, rtol=1e-12)
    finally:
        m.mskm_hier_destroy(hd)
        m.mskm_destroy(ctx)


@pytest.mark.parametrize("mode,top", [("fp64", 32900), ("fp32", 65700)])
def test_wide_groups(mode, top):
    """Levels of so many blocks that a workgroup takes four slices of right-hand sides (block counts that are
    no multiple of its sets of four, the last block not full): columns against their own solves."""
    import paper_2503_04914_amd as m

    R = 512
    h = synth.halton_hierarchy(sizes=[40, top // 5, top])
    base = [synth.fourier_target(4300 + r)(h.points) for r in range(4)]
    F = np.ascontiguousarray(np.stack([base[c % 4] * (1.0 + c) for c in range(R)], axis=1))
    ctx = m.mskm_create(0)
    hd = m.mskm_hier_create(ctx, h.points, h.offsets, h.delta, fp64=mode == "fp64", fp32=mode != "fp64")
    kw = dict(algorithm=m.MSKM_ALG_SEQUENTIAL, precond=m.MSKM_PRECOND_BLOCK_JACOBI)
    o = m.solve_opts(cg_rtol=1e-13, **kw) if mode == "fp64" else \
        m.solve_opts(precision=m.MSKM_PREC_FP32, cg_rtol=1e-5, target_rel_residual=1e-13, max_refine=20, **kw)
    try:
        A = np.zeros_like(F)
        r = m.mskm_solve(ctx, hd, F, A, o, nrhs=R)
        assert r.status == m.MSKM_OK, r.report
        assert m.mskm_residual(ctx, hd, A, F, nrhs=R).max() <= 1e-12
        for c in (0, 190, R - 1):
            a = np.zeros(len(F))
            assert m.mskm_solve(ctx, hd, np.ascontiguousarray(F[:, c]), a, o).status == m.MSKM_OK
            # two results, each within the repository's bar (1e-10 FP64, 1e-8 mixed)
            assert np.linalg.norm(A[:, c] - a) <= (2e-10 if mode == "fp64" else 2e-8) * np.linalg.norm(a)
    finally:
        m.mskm_hier_destroy(hd)
        m.mskm_destroy(ctx)
