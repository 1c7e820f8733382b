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
    spin = m.lib().mskm_test_spin
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


def _one_launch_and_launched(h, R, opts, sell=True, **store):
    import paper_2503_04914_amd as m

    spin, given_up, _ = _hooks(m)
    F = _targets(h, R)
    ctx = m.mskm_create(0)
    hd = m.mskm_hier_create(ctx, h.points, h.offsets, h.delta, **store)
    if sell:
        for prec in [p for p, k in ((m.MSKM_PREC_FP32, "fp32"), (m.MSKM_PREC_FP64, "fp64")) if store.get(k)]:
            m.mskm_set_spmv_width(hd, m.MSKM_OP_DIAG, prec, m.SELL_CODE)
    out = []
    try:
        for k in (SPIN, 0):
            print(f"[rounding] N={len(F)} R={R} spin limit {k}", flush=True)
            spin(ctx, k)
            A = np.zeros_like(F)
            r = m.mskm_solve(ctx, hd, F, A, opts(m), nrhs=R)
            out.append((A, r.report, r.status))
            assert (given_up(ctx) > 0) == (k == 0)
    finally:
        m.mskm_hier_destroy(hd)
        m.mskm_destroy(ctx)
    return out


# levels of one workgroup in every group of lanes, of two lanes and one lane a row, and past one sum a row (65,536 rows)
SIZES = {"one workgroup": [50, 250, 500, 1000], "two lanes a row": [257, 1030, 17001], "one lane a row": [4003, 64001],
         "entry order": [900, 90003]}


@pytest.mark.parametrize("sell", [True, False])  # the sliced product, or the default one of 8 lanes a row
@pytest.mark.parametrize("bj", [True, False])
@pytest.mark.parametrize("sizes", list(SIZES))
def test_one_launch_rounds_as_launched(sizes, bj, sell):
    import paper_2503_04914_amd as m

    h = synth.halton_hierarchy(sizes=SIZES[sizes])
    pc = m.MSKM_PRECOND_BLOCK_JACOBI if bj else m.MSKM_PRECOND_NONE
    (a, _, _), (b, _, _) = _one_launch_and_launched(h, 1, lambda m: _early(m, precond=pc), sell, fp64=False, fp32=True)
    _same_rounding(a, b)


@pytest.mark.parametrize("bj", [True, False])
@pytest.mark.parametrize("nu", [synth.NU_2D_40, 5.4])  # rows of about 40 and of 92 entries: one lane a row, two
def test_columns_round_as_launched(nu, bj):
    import paper_2503_04914_amd as m

    h = synth.halton_hierarchy(sizes=[257, 1030, 5003], nu=nu)
    pc = m.MSKM_PRECOND_BLOCK_JACOBI if bj else m.MSKM_PRECOND_NONE
    (a, _, _), (b, _, _) = _one_launch_and_launched(h, 21, lambda m: _early(m, precond=pc), fp64=False, fp32=True)
    _same_rounding(a, b)


def _level(n, nu=synth.NU_2D_40):
    return synth.halton_hierarchy(sizes=[n], nu=nu)


@pytest.mark.parametrize("R", [1, 3])
@pytest.mark.parametrize("rtol", [1e-7, 1e-12])
@pytest.mark.parametrize("n", [1365, 16385, 58000])
def test_fp32_preconditioned_tolerance(n, rtol, R):
    """One FP32 solve with block-Jacobi to tolerances below 1e-6, the default among them: as many iterations as
    the launched kernels need, give or take one (the stopping test on sums in another order)."""
    import paper_2503_04914_amd as m

    opts = lambda m: _mixed(m, cg_rtol=rtol, target_rel_residual=1e-3)  # noqa: E731  met after one round
    (_, ra, sa), (_, rb, sb) = _one_launch_and_launched(_level(n), R, opts, fp64=False, fp32=True)
    assert sa == sb == m.MSKM_OK
    assert ra["refine_steps"] == rb["refine_steps"] == 1
    assert abs(ra["cg_iters_total"] - rb["cg_iters_total"]) <= R, (ra, rb)
    assert ra["cg_iters_total"] < 1000 * R


@pytest.mark.parametrize("rtol", [1e-7, 1e-12])
@pytest.mark.parametrize("n", [65, 300])
def test_fp32_preconditioned_tolerance_one_workgroup(n, rtol):
    """Levels of one workgroup, which never give up: CG ends within as many iterations as unknowns, and the 1,365
    rows of the test above need about 120 to 1e-12."""
    import paper_2503_04914_amd as m

    ctx = m.mskm_create(0)
    h = _level(n)
    f = _targets(h, 1)
    hd = m.mskm_hier_create(ctx, h.points, h.offsets, h.delta, fp64=False, fp32=True)
    try:
        r = m.mskm_solve(ctx, hd, f, np.zeros_like(f), _mixed(m, cg_rtol=rtol, target_rel_residual=1e-3))
        assert r.status == m.MSKM_OK and r.report["refine_steps"] == 1
        assert r.report["cg_iters_total"] <= 200
    finally:
        m.mskm_hier_destroy(hd)
        m.mskm_destroy(ctx)


@pytest.mark.parametrize("R", [1, 2])
@pytest.mark.parametrize("nu,rtol", [(synth.NU_2D_40, 1e-15), (synth.NU_2D_40 * 1.22, 1e-14), (5.4, 1e-14)])
@pytest.mark.parametrize("n", [341, 1025, 4225, 20000])
def test_fp64_preconditioned_tolerance(n, nu, rtol, R):
    """FP64 with block-Jacobi on rows of about 40, 60 and 92 entries, to where the launched kernels still stop by
    themselves (a level that breaks off or runs to its cap is reported as not converged)."""
    import paper_2503_04914_amd as m

    ctx = m.mskm_create(0)
    h = _level(n, nu)
    F = _targets(h, R)
    hd = m.mskm_hier_create(ctx, h.points, h.offsets, h.delta, fp64=True, fp32=False)
    try:
        r = m.mskm_solve(ctx, hd, F, np.zeros_like(F),
                         m.solve_opts(cg_rtol=rtol, algorithm=m.MSKM_ALG_SEQUENTIAL,
                                      precond=m.MSKM_PRECOND_BLOCK_JACOBI), nrhs=R)
        assert r.status == m.MSKM_OK, r.report
    finally:
        m.mskm_hier_destroy(hd)
        m.mskm_destroy(ctx)


@pytest.mark.parametrize("sell", [True, False])
@pytest.mark.parametrize("bj", [True, False])
@pytest.mark.parametrize("case", ["halton", "uniform3d", "wide rows", "few wide rows", "small wide levels"])
def test_large_levels_round_as_launched(case, bj, sell):
    """Levels whose matrix does not fit the registers: many rows, and rows of about 180 entries on levels past and
    below the rows (65,536) that the launched kernels split a row's sum in two for, and the rows (1,024) that they
    solve in one workgroup."""
    import paper_2503_04914_amd as m

    h = {"halton": lambda: synth.halton_hierarchy(sizes=[1000, 256 * 1024 + 77]),
         "uniform3d": lambda: synth.uniform3d_hierarchy(2, n0=20000),
         "wide rows": lambda: synth.halton_hierarchy(sizes=[5003, 70001], nu=7.5),
         "few wide rows": lambda: synth.halton_hierarchy(sizes=[1025, 9001], nu=7.5),
         "small wide levels": lambda: synth.halton_hierarchy(sizes=[300, 900], nu=7.5)}[case]()
    pc = m.MSKM_PRECOND_BLOCK_JACOBI if bj else m.MSKM_PRECOND_NONE
    (a, _, _), (b, _, _) = _one_launch_and_launched(h, 1, lambda m: _early(m, precond=pc), sell, fp64=False, fp32=True)
    _same_rounding(a, b)
