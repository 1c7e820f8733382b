"""Several contexts on one GPU, each with a thread and a stream of its own, solving at the same time: the one-launch CG
of one waits for that of another instead of sharing the GPU with it."""
import ctypes
import threading

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_contexts_in_threads():
    import paper_2503_04914_amd as m

    given_up = m.lib().mskm_test_given_up
    given_up.argtypes, given_up.restype = [ctypes.c_void_p], ctypes.c_int64
    cases = [([300, 1200, 4800], 1), ([1000, 90003], 1), ([257, 5003], 3)]
    kw = dict(precision=m.MSKM_PREC_FP32, algorithm=m.MSKM_ALG_SEQUENTIAL, cg_rtol=1e-5, target_rel_residual=1e-12,
              max_refine=20, precond=m.MSKM_PRECOND_BLOCK_JACOBI)
    data = []
    for sizes, R in cases:
        h = synth.halton_hierarchy(sizes=sizes)
        F = np.ascontiguousarray(np.stack([synth.fourier_target(6300 + r)(h.points) for r in range(R)], axis=1))
        data.append((h, F[:, 0].copy() if R == 1 else F, R))

    def solve(k, times):
        h, F, R = data[k]
        ctx = m.mskm_create(0)
        hd = m.mskm_hier_create(ctx, h.points, h.offsets, h.delta, fp64=False, fp32=True)
        out = []
        try:
            for _ in range(times):
                a = np.zeros_like(F)
                r = m.mskm_solve(ctx, hd, F, a, m.solve_opts(**kw), nrhs=R)
                assert r.status == m.MSKM_OK, r.report
                out.append(a)
            return out, given_up(ctx)
        finally:
            m.mskm_hier_destroy(hd)
            m.mskm_destroy(ctx)

    want = [solve(k, 1)[0][0] for k in range(len(data))]
    got = [None] * len(data)

    def work(k):
        got[k] = solve(k, 20)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(data))]
    print("[contexts] three threads", flush=True)
    for t in threads:
        t.start()
    for t in threads:
        t.join(100)
    for k, g in enumerate(got):
        assert g is not None, k
        assert g[1] == 0
        for a in g[0]:
            assert np.array_equal(a, want[k])
