"""The one-launch CG rounds as the launched kernels do and reaches the tolerances they reach.

Rounding is compared on the FP32 solution after ten iterations. Kernels that add a row's products in another order
round most entries differently by then. The sums over a level are added in FP64 in another order in the one-launch
CG and on the tiles, which changes them by about 1e-15 of their value and an FP32 entry's rounding once in some 1e8
entries; one such entry changes the next steps by up to 1e-10 of their length, the rounding of up to 1e-10 / 6e-8 of
all entries. SHARE, ten times that, tells the two apart.
"""
import ctypes

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

SPIN, SHARE = 1 << 15, 0.02


def _hooks(m):
    spin = getattr(m.lib(), "_ZN4mskm16cg_grid_set_spinEP8mskm_ctxi")
    spin.argtypes, spin.restype = [ctypes.c_void_p, ctypes.c_int], None
    given_up, limits = m.lib().mskm_test_given_up, m.lib().mskm_test_limits
    given_up.argtypes, given_up.restype = [ctypes.c_void_p], ctypes.c_int64
    limits.argtypes, limits.restype = [ctypes.c_void_p, ctypes.c_uint64, ctypes.c_uint64], None
    return spin, given_up, limits


def _targets(h, R):
    f = [synth.fourier_target(5300 + r, h.dim)(h.points) for r in range(R)]
    return f[0] if R == 1 else np.ascontiguousarray(np.stack(f, axis=1))


def _mixed(m, **kw):
    return m.solve_opts(**dict(dict(precision=m.MSKM_PREC_FP32, algorithm=m.MSKM_ALG_SEQUENTIAL, cg_rtol=1e-5,
                                    target_rel_residual=1e-13, max_refine=20,
                                    precond=m.MSKM_PRECOND_BLOCK_JACOBI), **kw))


def _early(m, **kw):
    return _mixed(m, **dict(dict(max_cg_iters=10, max_refine=1), **kw))


def _same_rounding(a, b):
    assert np.all(np.isfinite(a)) and np.any(a)
    assert np.mean(a != b) <= SHARE, np.mean(a != b)


@pytest.mark.parametrize("R", [17, 64, 256])
def test_tiles_round_as_rows(R):
    """On the tiles and, without memory for them, row by row."""
    import paper_2503_04914_amd as m

    spin, _, limits = _hooks(m)
    h = synth.halton_hierarchy(sizes=[301, 5003, 80011])
    F = _targets(h, R)
    ctx = m.mskm_create(0)
    out = []
    try:
        spin(ctx, 0)  # launched kernels on every level
        for rows in (False, True):
            hd = m.mskm_hier_create(ctx, h.points, h.offsets, h.delta, fp64=False, fp32=True)
            # one right-hand side first: the preconditioner
            assert m.mskm_solve(ctx, hd, np.ascontiguousarray(F[:, 0]), np.zeros(len(F)), _mixed(m)).status == m.MSKM_OK
            print(f"[rounding] tiles, R={R}, rows={rows}", flush=True)
            limits(ctx, 1 if rows else 0, 0)
            A = np.zeros_like(F)
            m.mskm_solve(ctx, hd, F, A, _early(m), nrhs=R)
            limits(ctx, 0, 0)
            m.mskm_hier_destroy(hd)
            out.append(A)
    finally:
        m.mskm_destroy(ctx)
    _same_rounding(*out)
