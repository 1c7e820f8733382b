"""Queries at the edges of the rule that sorts them by cells: the same values, bit for bit, as in calls too small for it."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq", [131071, 131072, 200003])
@pytest.mark.parametrize("case", ["below an L2", "halton", "one level", "uniform3d"])
def test_order_changes_no_value(case, nq):
    import paper_2503_04914_amd as m

    h = {"below an L2": lambda: synth.halton_hierarchy(sizes=[5000, 150001]),   # 24 bytes a point: 3.7 MB
         "halton": lambda: synth.halton_hierarchy(sizes=[3, 4097, 200001]),     # 4.9 MB
         "one level": lambda: synth.halton_hierarchy(sizes=[220001]),
         "uniform3d": lambda: synth.uniform3d_hierarchy(1, n0=150001)}[case]()  # 32 bytes a point: 4.8 MB
    rng = np.random.default_rng(22)
    A, Q = rng.standard_normal((h.n_total, 3)), rng.uniform(-0.1, 1.1, (nq, h.dim))
    ctx = m.mskm_create(0)
    hd = m.mskm_hier_create(ctx, h.points, h.offsets, h.delta)
    try:
        whole = np.empty((nq, 3))
        m.mskm_evaluate(ctx, hd, A, Q, whole, nrhs=3)
        at = 0
        for q in np.array_split(Q, 3):
            q = np.ascontiguousarray(q)
            part = np.empty((len(q), 3))
            m.mskm_evaluate(ctx, hd, A, q, part, nrhs=3)
            assert np.array_equal(part, whole[at:at + len(q)])
            at += len(q)
        assert np.all(np.isfinite(whole))
    finally:
        m.mskm_hier_destroy(hd)
        m.mskm_destroy(ctx)
