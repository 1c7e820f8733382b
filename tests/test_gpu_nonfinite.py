"""Infinite and undefined data among many right-hand sides."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("nrhs", [2, 16, 33])
def test_residuals_of_non_finite_columns(nrhs, fp32):
    """Residuals at once, on the tiles, against one by one: an infinite coefficient or value gives inf where its
    products do not cancel, and the other columns are not touched."""
    import paper_2503_04914_amd as m

    h = synth.halton_hierarchy(sizes=[60, 300, 5003])
    F = np.ascontiguousarray(np.stack([synth.fourier_target(6100 + r)(h.points) for r in range(nrhs)], axis=1))
    A = np.random.default_rng(61).standard_normal(F.shape)
    ctx = m.mskm_create(0)
    hd = m.mskm_hier_create(ctx, h.points, h.offsets, h.delta, fp64=not fp32, fp32=fp32)
    try:
        m.mskm_residual(ctx, hd, np.ascontiguousarray(np.repeat(A, 16, axis=1)[:, :16]),
                        np.ascontiguousarray(np.repeat(F, 16, axis=1)[:, :16]), nrhs=16)  # builds the tiles
        plain = m.mskm_residual(ctx, hd, A, F, nrhs=nrhs)
        for name, x, at, v in (("coefficient", A, 4000, np.inf), ("coefficient", A, 100, -np.inf),
                               ("coefficient", A, 5, np.nan), ("value", F, 200, np.inf), ("coefficient", A, 4001, 1e200)):
            B = x.copy()
            B[at, 1] = v
            a, f = (B, F) if x is A else (A, B)
            got = m.mskm_residual(ctx, hd, a, f, nrhs=nrhs)
            one = [float(np.ravel(m.mskm_residual(ctx, hd, np.ascontiguousarray(a[:, c]),
                                                  np.ascontiguousarray(f[:, c])))[0]) for c in (0, 1)]
            print(f"[non-finite] {name} {v} at {at}: {np.ravel(got)[1]} (alone {one[1]})", flush=True)
            # the same FP64 products in another order: 1e-12 of residuals of order one
            np.testing.assert_allclose(np.ravel(got)[:2], one, rtol=1e-12)
            keep = [c for c in range(nrhs) if c != 1]
            np.testing.assert_allclose(np.ravel(got)[keep], np.ravel(plain)[keep], rtol=1e-12)
    finally:
        m.mskm_hier_destroy(hd)
        m.mskm_destroy(ctx)


@pytest.mark.parametrize("mixed", [False, True])
def test_solves_beside_non_finite_columns(mixed):
    """Columns of a device array (whose values are not looked at beforehand) with an infinite or undefined value are
    reported, the others' solutions are bit for bit those without it, and the bad columns' coefficients are finite."""
    import torch

    import paper_2503_04914_amd as m

    h = synth.halton_hierarchy(sizes=[60, 300, 1200, 20011])
    F = np.ascontiguousarray(np.stack([synth.fourier_target(6200 + r)(h.points) for r in range(17)], axis=1))
    B = F.copy()
    B[100, 2], B[1700, 5] = np.inf, np.nan
    ctx = m.mskm_create(0)
    hd = m.mskm_hier_create(ctx, h.points, h.offsets, h.delta, fp64=not mixed, fp32=mixed)
    kw = dict(algorithm=m.MSKM_ALG_SEQUENTIAL, precond=m.MSKM_PRECOND_BLOCK_JACOBI)
    o = m.solve_opts(precision=m.MSKM_PREC_FP32, cg_rtol=1e-5, target_rel_residual=1e-30, max_refine=1, **kw) \
        if mixed else m.solve_opts(cg_rtol=1e-12, **kw)
    try:
        dev = [torch.from_numpy(x).to("cuda:0") for x in (F, B, F, F)]
        torch.cuda.synchronize()
        m.mskm_solve(ctx, hd, dev[0], dev[2], o, nrhs=17)
        assert m.mskm_solve(ctx, hd, dev[1], dev[3], o, nrhs=17).status == m.MSKM_ENOCONV
        a, b = dev[2].cpu().numpy(), dev[3].cpu().numpy()
        keep = [c for c in range(17) if c not in (2, 5)]
        assert np.array_equal(a[:, keep], b[:, keep])
        assert np.all(np.isfinite(b))
    finally:
        m.mskm_hier_destroy(hd)
        m.mskm_destroy(ctx)
