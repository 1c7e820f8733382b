"""The ways without the one-launch CG and without the tiles: a persistent
launch that gives up is counted and its levels are solved by launched kernels;
without memory for tiles the many-right-hand-side products go row by row.
"""
import ctypes

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

SPIN = 1 << 15  # polls of a wait


def _hooks(m):
    spin = m.lib().mskm_test_spin
    spin.argtypes, spin.restype = [ctypes.c_void_p, ctypes.c_int], None
    given_up, limits = m.lib().mskm_test_given_up, m.lib().mskm_test_limits
    given_up.argtypes, given_up.restype = [ctypes.c_void_p], ctypes.c_int64
    limits.argtypes, limits.restype = [ctypes.c_void_p, ctypes.c_uint64, ctypes.c_uint64], None
    return spin, given_up, limits


def _opts(m, mixed, **kw):
    kw = dict(dict(algorithm=m.MSKM_ALG_SEQUENTIAL, precond=m.MSKM_PRECOND_BLOCK_JACOBI), **kw)
    return m.solve_opts(precision=m.MSKM_PREC_FP32, cg_rtol=1e-5, target_rel_residual=1e-13, max_refine=20, **kw) \
        if mixed else m.solve_opts(cg_rtol=1e-13, **kw)


def _targets(h, R):
    return np.ascontiguousarray(np.stack([synth.fourier_target(5100 + r)(h.points) for r in range(R)], axis=1))


@pytest.mark.parametrize("R", [1, 3])
@pytest.mark.parametrize("mixed", [False, True])
def test_given_up_launches_are_counted(mixed, R):
    import paper_2503_04914_amd as m

    spin, given_up, _ = _hooks(m)
    h = synth.halton_hierarchy(sizes=[300, 1200, 4800])
    F = _targets(h, R)
    ctx = m.mskm_create(0)
    hd = m.mskm_hier_create(ctx, h.points, h.offsets, h.delta, fp64=True, fp32=mixed)
    try:
        a, b = np.zeros_like(F), np.zeros_like(F)
        assert m.mskm_solve(ctx, hd, F, a, _opts(m, mixed), nrhs=R).status == m.MSKM_OK
        assert given_up(ctx) == 0
        print("[ways back] spin limit 0", flush=True)
        spin(ctx, 0)
        assert m.mskm_solve(ctx, hd, F, b, _opts(m, mixed), nrhs=R).status == m.MSKM_OK
        assert given_up(ctx) > 0
        spin(ctx, SPIN)
        n = given_up(ctx)
        assert m.mskm_solve(ctx, hd, F, b, _opts(m, mixed), nrhs=R).status == m.MSKM_OK
        assert given_up(ctx) == n
        assert np.array_equal(a, b)
    finally:
        m.mskm_hier_destroy(hd)
        m.mskm_destroy(ctx)


def _tiles_and_rows(mixed, R, sizes):
    """Solutions and residuals on the tiles and, on a second hierarchy without memory for them, row by row."""
    import paper_2503_04914_amd as m

    _, _, limits = _hooks(m)
    h = synth.halton_hierarchy(sizes=sizes)
    F = _targets(h, R)
    ctx = m.mskm_create(0)
    out = []
    try:
        for rows in (False, True):
            hd = m.mskm_hier_create(ctx, h.points, h.offsets, h.delta, fp64=not mixed, fp32=mixed)
            A, one = np.zeros_like(F), np.zeros(len(F))
            # one right-hand side first: the preconditioner and the plans of the one-launch CG
            assert m.mskm_solve(ctx, hd, np.ascontiguousarray(F[:, 0]), one, _opts(m, mixed)).status == m.MSKM_OK
            print(f"[tiles] rows={rows} R={R} mixed={mixed}", flush=True)
            if rows:
                limits(ctx, 1, 0)
            assert m.mskm_solve(ctx, hd, F, A, _opts(m, mixed), nrhs=R).status == m.MSKM_OK
            res = m.mskm_residual(ctx, hd, A, F, nrhs=R)
            limits(ctx, 0, 0)
            m.mskm_hier_destroy(hd)
            out.append((A, res))
    finally:
        m.mskm_destroy(ctx)
    return out


@pytest.mark.parametrize("R", [2, 17, 64])
@pytest.mark.parametrize("mixed", [False, True])
def test_row_by_row_products(mixed, R):
    """The repository's bars for two results of one system: 1e-10 each in FP64, 1e-8 refined mixed."""
    (A, ra), (B, rb) = _tiles_and_rows(mixed, R, [60, 301, 1204, 20011])
    assert ra.max() <= 1e-12 and rb.max() <= 1e-12
    assert np.linalg.norm(A - B) <= (2e-8 if mixed else 2e-10) * np.linalg.norm(A)


@pytest.mark.parametrize("R", [1, 3])
def test_a_give_up_is_remembered(R):
    """A launch that gives up is tried once: the launches behind it, the rounds of that solve and the next solves
    go without (their count stays), and the results are those of the launched kernels."""
    import paper_2503_04914_amd as m

    spin, given_up, _ = _hooks(m)
    h = synth.halton_hierarchy(sizes=[300, 1200, 4800, 140001])  # 4 depths, one past the registers and one launch
    F = _targets(h, R)
    ctx = m.mskm_create(0)
    hd = m.mskm_hier_create(ctx, h.points, h.offsets, h.delta, fp64=True, fp32=True)
    out = []
    try:
        for mixed in (True, False):
            print(f"[ways back] remembered, R={R} mixed={mixed}", flush=True)
            spin(ctx, 0)
            n = given_up(ctx)
            a, b, c = np.zeros_like(F), np.zeros_like(F), np.zeros_like(F)
            r = m.mskm_solve(ctx, hd, F, a, _opts(m, mixed), nrhs=R)
            assert r.status == m.MSKM_OK
            if mixed:
                assert r.report["refine_steps"] > 1
            assert n < given_up(ctx) <= n + h.levels
            n = given_up(ctx)
            assert m.mskm_solve(ctx, hd, F, b, _opts(m, mixed), nrhs=R).status == m.MSKM_OK
            assert given_up(ctx) == n
            if R == 1:  # (of several, levels of one workgroup, which cannot give up, were solved in one launch in a)
                assert np.array_equal(a, b)
            spin(ctx, SPIN)
            assert m.mskm_solve(ctx, hd, F, c, _opts(m, mixed), nrhs=R).status == m.MSKM_OK
            assert given_up(ctx) == n
            out.append((a, c))
    finally:
        m.mskm_hier_destroy(hd)
        m.mskm_destroy(ctx)
    for (a, c), bar in zip(out, (2e-8, 2e-10)):  # two results within the repository's bars, 1e-8 mixed and 1e-10 FP64
        assert np.linalg.norm(a - c) <= bar * np.linalg.norm(c)


def test_no_scratch_memory():
    """Without memory for their scratch blocks, an evaluation goes one right-hand side at a time (with and without
    the solver's vectors) and a solve of several right-hand sides one after the other."""
    import paper_2503_04914_amd as m

    _, _, limits = _hooks(m)
    h = synth.halton_hierarchy(sizes=[300, 5003, 200001])
    F = _targets(h, 5)
    q = synth.uniform01(5200, 0, 2 * 140001).reshape(-1, 2)  # as many points and queries as are sorted otherwise
    ctx = m.mskm_create(0)
    hd = m.mskm_hier_create(ctx, h.points, h.offsets, h.delta, fp64=True, fp32=True)
    o = _opts(m, True)
    try:
        for solved in (False, True):
            for R in (1, 2, 5):
                x = np.ascontiguousarray(F[:, :R])
                v, w = np.zeros((len(q), R)), np.zeros((len(q), R))
                m.mskm_evaluate(ctx, hd, x, q, v, nrhs=R)
                limits(ctx, 0, 1)
                m.mskm_evaluate(ctx, hd, x, q, w, nrhs=R)
                limits(ctx, 0, 0)
                # sums of about 150 terms in FP64
                assert np.abs(v - w).max() <= 1e-12 * np.abs(v).max()
            a, b = np.zeros((len(F), 2)), np.zeros(len(F))
            limits(ctx, 0, 1)
            r = m.mskm_solve(ctx, hd, np.ascontiguousarray(F[:, :2]), a, o, nrhs=2)
            limits(ctx, 0, 0)
            assert r.status == m.MSKM_OK
            for c in range(2):
                assert m.mskm_solve(ctx, hd, np.ascontiguousarray(F[:, c]), b, o).status == m.MSKM_OK
                assert np.array_equal(a[:, c], b)
    finally:
        m.mskm_hier_destroy(hd)
        m.mskm_destroy(ctx)


@pytest.mark.parametrize("cap", [1, 8 << 20, 32 << 30])
def test_block_cache(cap):
    """Hierarchies of changing sizes on a block cache of nothing, of less than one of them, and of the ordinary
    size: the same coefficients, and no more bytes held than the cap."""
    import paper_2503_04914_amd as m

    cache = m.lib().mskm_test_cache
    cache.argtypes, cache.restype = [ctypes.c_void_p, ctypes.c_uint64], ctypes.c_uint64
    ctx = m.mskm_create(0)
    first = {}
    try:
        cache(ctx, cap)
        for n in (5000, 20011, 5000, 20480, 5003, 20011):
            h = synth.halton_hierarchy(sizes=[n // 16, n // 4, n])
            F = _targets(h, 2)
            a, A = np.zeros(len(F)), np.zeros_like(F)
            hd = m.mskm_hier_create(ctx, h.points, h.offsets, h.delta, fp64=False, fp32=True, sliced_lower=True)
            assert m.mskm_solve(ctx, hd, np.ascontiguousarray(F[:, 0]), a, _opts(m, True)).status == m.MSKM_OK
            assert m.mskm_solve(ctx, hd, F, A, _opts(m, True), nrhs=2).status == m.MSKM_OK
            m.mskm_hier_destroy(hd)
            held = cache(ctx, 0)
            assert held <= cap and (held > 0 or cap == 1)
            if n in first:
                assert np.array_equal(a, first[n][0]) and np.array_equal(A, first[n][1])
            first[n] = a, A
    finally:
        m.mskm_destroy(ctx)
