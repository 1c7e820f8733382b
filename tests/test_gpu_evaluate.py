"""Evaluation of the approximant: queries sorted by cells against the same
queries in small calls (unsorted), several right-hand sides at once against one
at a time, queries outside the points' box, single-cell levels, 3-D; and a
sample against the plain sum.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _h(case):
    if case == "halton":
        return synth.halton_hierarchy(sizes=[3, 70, 4097, 140001])
    return synth.uniform3d_hierarchy(3, n0=2100)  # 2,100 .. 134,400 points


@pytest.mark.parametrize("case", ["halton", "uniform3d"])
def test_orders_and_widths_agree(case):
    import paper_2503_04914_amd as m

    h = _h(case)
    rng = np.random.default_rng(21)
    A = rng.standard_normal((h.n_total, 5))
    Q = rng.uniform(-0.2, 1.2, (40001, h.dim))
    ctx = m.mskm_create(0)
    hd = m.mskm_hier_create(ctx, h.points, h.offsets, h.delta)

    def value(a, q):
        a, q = np.ascontiguousarray(a), np.ascontiguousarray(q)
        nrhs = 1 if a.ndim == 1 else a.shape[1]
        out = np.empty((len(q), nrhs))
        m.mskm_evaluate(ctx, hd, a, q, out, nrhs=nrhs)
        return out

    try:
        one = np.concatenate([value(A[:, r], Q) for r in range(5)], axis=1)  # sorted
        parts = np.concatenate([value(A[:, 0], q) for q in np.array_split(Q, 3)])  # unsorted: below the sort's size
        assert np.array_equal(parts[:, 0], one[:, 0])  # the order of the queries changes no sum
        for nrhs in (2, 3, 4, 5):
            assert np.array_equal(value(A[:, :nrhs], Q), one[:, :nrhs])
        assert value(A[:, 0], Q[:0]).shape == (0, 1)
        sel = rng.choice(len(Q), 50, replace=False)
        ref = np.zeros(50)
        for l in range(h.levels):
            x, a = h.level_points(l), A[h.offsets[l]:h.offsets[l + 1], 0]
            r = np.sqrt(((Q[sel][:, None, :] - x[None]) ** 2).sum(axis=2)) / h.delta[l]
            ref += (np.maximum(1.0 - r, 0.0) ** 4 * (4.0 * r + 1.0)) @ a
        # FP64 sums of at most a few hundred terms of order one
        assert np.max(np.abs(one[sel, 0] - ref)) <= 1e-12 * max(1.0, np.max(np.abs(ref)))
    finally:
        m.mskm_hier_destroy(hd)
        m.mskm_destroy(ctx)
