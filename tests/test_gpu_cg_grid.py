"""The CG of middle-sized levels in one launch of workgroups that exchange
their sums and direction entries on the device: sizes at the edges of its
workgroups (256 or 512 rows), rows longer than its registers hold, levels past
its range, and its way back to the launched kernels when a wait is given up.
"""
import ctypes

import numpy as np
import pytest

import oracle
import synth
from oracle import multiscale as ms

pytestmark = pytest.mark.gpu


def _hier(top, nu=synth.NU_2D_40, dim=2):
    if dim == 3:
        pts = synth.uniform01(2100 + top, 0, 3 * top).reshape(-1, 3)
        return pts, np.array([0, top], dtype=np.int64), np.array([nu * top ** (-1.0 / 3.0)])
    sizes = [max(top // 4, 1), top]
    pts = synth.halton(top)
    return (np.concatenate([pts[:n] for n in sizes]), np.cumsum([0] + sizes).astype(np.int64),
            np.array([nu * n ** -0.5 for n in sizes]))


def _check(m, ctx, pts, offs, delta, mixed, bj):
    hd = m.mskm_hier_create(ctx, pts, offs, delta, fp64=True, fp32=mixed)
    f = synth.fourier_target(1300, dim=pts.shape[1])(pts)
    kw = dict(precond=m.MSKM_PRECOND_BLOCK_JACOBI if bj else m.MSKM_PRECOND_NONE, algorithm=m.MSKM_ALG_SEQUENTIAL)
    o = m.solve_opts(precision=m.MSKM_PREC_FP32, cg_rtol=1e-4, target_rel_residual=1e-13, max_refine=20, **kw) if mixed \
        else m.solve_opts(cg_rtol=1e-13, **kw)
    try:
        a, b = np.zeros_like(f), np.zeros_like(f)
        r = m.mskm_solve(ctx, hd, f, a, o)
        assert r.status == m.MSKM_OK, r.report
        assert m.mskm_solve(ctx, hd, f, b, o).status == m.MSKM_OK
        assert np.array_equal(a, b)  # fixed-order sums
        assert r.report["cg_iters_total"] > 0
    finally:
        m.mskm_hier_destroy(hd)
    ref = oracle.sequential_solve(ms.assemble(pts, offs, delta), f)
    # the repository's bars: FP64 coefficients 1e-10, refined mixed ones 1e-8
    for l in range(len(delta)):
        sl = slice(offs[l], offs[l + 1])
        assert np.linalg.norm(a[sl] - ref[sl]) <= (1e-8 if mixed else 1e-10) * np.linalg.norm(ref[sl])


@pytest.mark.parametrize("bj", [False, True])
@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("top", [1, 255, 256, 257, 1025, 4099])
def test_level_sizes(top, mixed, bj):
    import paper_2503_04914_amd as m

    ctx = m.mskm_create(0)
    try:
        _check(m, ctx, *_hier(top), mixed, bj)
    finally:
        m.mskm_destroy(ctx)


@pytest.mark.parametrize("bj", [False, True])
@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("top", [300, 511, 512, 513])
def test_one_workgroup_levels(top, mixed, bj):
    import paper_2503_04914_amd as m

    ctx = m.mskm_create(0)
    try:
        _check(m, ctx, *_hier(top), mixed, bj)
    finally:
        m.mskm_destroy(ctx)


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("case", ["rows of about 100", "rows past 128", "3-D"])
def test_row_lengths(case, mixed):
    """Rows that need more registers, too many, and a 3-D level with long rows and halos."""
    import paper_2503_04914_amd as m

    nu = {"rows of about 100": 5.4, "rows past 128": 7.5, "3-D": synth.NU_3D_60}[case]
    ctx = m.mskm_create(0)
    try:
        _check(m, ctx, *_hier(2300, nu, 3 if case == "3-D" else 2), mixed, True)
    finally:
        m.mskm_destroy(ctx)


@pytest.mark.parametrize("algorithm", ["monolithic", "sequential"])
def test_all_level_kinds_agree(algorithm):
    """Levels of one workgroup, of 256- and 512-row workgroups and past the
    range together: FP64 coefficients equal to those of the launched kernels
    (a spin limit of 0 gives every wait up at once), which also takes the way
    back."""
    import paper_2503_04914_amd as m

    h = synth.halton_hierarchy(sizes=[60, 1030, 17001, 66001, 140003])
    f = synth.fourier_target(1301)(h.points)
    set_spin = getattr(m.lib(), "_ZN4mskm16cg_grid_set_spinEP8mskm_ctxi")
    set_spin.argtypes, set_spin.restype = [ctypes.c_void_p, ctypes.c_int], None
    ctx = m.mskm_create(0)
    hd = m.mskm_hier_create(ctx, h.points, h.offsets, h.delta)
    alg = m.MSKM_ALG_MONOLITHIC if algorithm == "monolithic" else m.MSKM_ALG_SEQUENTIAL
    o = m.solve_opts(cg_rtol=1e-13, algorithm=alg)
    try:
        out = []
        for spin in (1 << 15, 0, 1 << 15):
            print(f"[grid] spin limit {spin}", flush=True)
            set_spin(ctx, spin)
            a = np.zeros_like(f)
            r = m.mskm_solve(ctx, hd, f, a, o)
            assert r.status == m.MSKM_OK, r.report
            assert r.report["rel_residual"] <= 1e-12
            out.append(a)
        assert np.array_equal(out[0], out[2])
        assert np.linalg.norm(out[1] - out[0]) <= 1e-10 * np.linalg.norm(out[0])
    finally:
        m.mskm_hier_destroy(hd)
        m.mskm_destroy(ctx)


@pytest.mark.parametrize("bj", [False, True])
@pytest.mark.parametrize("case", ["one slot past a multiple of 512 rows", "uneven levels of one depth", "3-D", "wide rows"])
def test_large_fp32_levels(case, bj):
    """The FP32 form for levels past the registers: its coefficients (refined to 1e-13) equal to those of
    the launched kernels (spin limit 0), and repeats bit for bit."""
    import paper_2503_04914_amd as m

    if case == "3-D":
        h = synth.uniform3d_hierarchy(2, n0=20000)  # 20,000 and 160,000 points
        hs = [h]
    elif case == "uneven levels of one depth":
        hs = [synth.halton_hierarchy(sizes=s, start=1 + 500000 * k)
              for k, s in enumerate(([50, 150001], [1200, 3001], [400, 90007]))]
    elif case == "wide rows":
        hs = [synth.halton_hierarchy(sizes=[5000, 140001], nu=5.4)]  # about 92 entries a row
    else:
        hs = [synth.halton_hierarchy(sizes=[1000, 256 * 1024 + 77])]
    set_spin = getattr(m.lib(), "_ZN4mskm16cg_grid_set_spinEP8mskm_ctxi")
    set_spin.argtypes, set_spin.restype = [ctypes.c_void_p, ctypes.c_int], None
    f = np.concatenate([synth.fourier_target(1400 + k, h.dim)(h.points) for k, h in enumerate(hs)])
    ctx = m.mskm_create(0)
    hd = m.mskm_hier_create_batch(ctx, [(h.points, h.offsets, h.delta) for h in hs], fp64=False, fp32=True)
    o = m.solve_opts(precision=m.MSKM_PREC_FP32, algorithm=m.MSKM_ALG_SEQUENTIAL, cg_rtol=1e-5, max_refine=20,
                     target_rel_residual=1e-13,
                     precond=m.MSKM_PRECOND_BLOCK_JACOBI if bj else m.MSKM_PRECOND_NONE)
    try:
        out = []
        for spin in (1 << 15, 0, 1 << 15):
            print(f"[stream] spin limit {spin}", flush=True)
            set_spin(ctx, spin)
            a = np.zeros_like(f)
            r = m.mskm_solve(ctx, hd, f, a, o)
            assert r.status == m.MSKM_OK, r.report
            out.append(a)
        assert np.array_equal(out[0], out[2])
        # both within the repository's bar for refined mixed coefficients (1e-8)
        assert np.linalg.norm(out[1] - out[0]) <= 2e-8 * np.linalg.norm(out[0])
    finally:
        m.mskm_hier_destroy(hd)
        m.mskm_destroy(ctx)


@pytest.mark.parametrize("bj", [False, True])
@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("R", [3, 33, 300])
def test_columns(R, mixed, bj):
    """Many right-hand sides on small levels (in one launch, in several, and too many for it): every column's
    residual, columns equal to their own solves, and the way back to the launched kernels (spin limit 0)."""
    import paper_2503_04914_amd as m

    h = synth.halton_hierarchy(sizes=[60, 300, 1200, 4800])
    F = np.ascontiguousarray(np.stack([synth.fourier_target(1500 + r)(h.points) for r in range(R)], axis=1))
    F[:, 1] = 0.0
    set_spin = getattr(m.lib(), "_ZN4mskm16cg_grid_set_spinEP8mskm_ctxi")
    set_spin.argtypes, set_spin.restype = [ctypes.c_void_p, ctypes.c_int], None
    kw = dict(algorithm=m.MSKM_ALG_SEQUENTIAL, precond=m.MSKM_PRECOND_BLOCK_JACOBI if bj else m.MSKM_PRECOND_NONE)
    o = m.solve_opts(precision=m.MSKM_PREC_FP32, cg_rtol=1e-5, target_rel_residual=1e-13, max_refine=20, **kw) \
        if mixed else m.solve_opts(cg_rtol=1e-13, **kw)
    bar = 2e-8 if mixed else 2e-10  # two results, each within the repository's bar (1e-8 mixed, 1e-10 FP64)
    ctx = m.mskm_create(0)
    hd = m.mskm_hier_create(ctx, h.points, h.offsets, h.delta, fp64=True, fp32=mixed)
    try:
        out = []
        for spin in (1 << 15, 0, 1 << 15):
            print(f"[columns] spin limit {spin}", flush=True)
            set_spin(ctx, spin)
            A = np.zeros_like(F)
            r = m.mskm_solve(ctx, hd, F, A, o, nrhs=R)
            assert r.status == m.MSKM_OK, r.report
            assert m.mskm_residual(ctx, hd, A, F, nrhs=R).max() <= 1e-12
            assert np.all(A[:, 1] == 0.0)
            out.append(A)
        assert np.array_equal(out[0], out[2])
        assert np.linalg.norm(out[1] - out[0]) <= bar * np.linalg.norm(out[0])
        for c in {0, R // 2, R - 1}:
            a = np.zeros(len(F))
            assert m.mskm_solve(ctx, hd, np.ascontiguousarray(F[:, c]), a, o).status == m.MSKM_OK
            assert np.linalg.norm(out[0][:, c] - a) <= bar * np.linalg.norm(a)
    finally:
        m.mskm_hier_destroy(hd)
        m.mskm_destroy(ctx)
