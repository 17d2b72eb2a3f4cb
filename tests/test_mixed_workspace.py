"""A caller's workspace for the mixed Newton step: tm_workspace_bytes covers the FP64 updates of few systems, so that
a context given that much takes the launches of one that allocates for itself (bitwise), and a workspace of the
float32 size still serves (more launches, or float32 updates: the mixed step's 1e-8 bar).
"""
import ctypes
import sys

import numpy as np
import pytest
import torch

import synth
from paper_1809_05608_amd import tm


def _slot(p, bytes_per):
    nt = (p.n_groups + 3) // 4 * 4
    return p.n_zones * nt * (nt + 1) * bytes_per


def test_bytes_cover_the_fp64_updates_of_few_systems():
    lib = tm.load_library()
    for R, few in ((10, True), (1024, True), (1025, False)):
        p = tm.make_problem(4, R, 540, 13, 1.0, precision=tm.PREC_MIXED)
        for b in (1, 7, 4 * R):
            least = (b + 15) * _slot(p, 4)
            want = max(least, (b + 1) * _slot(p, 8)) if few else least
            assert lib.tm_workspace_bytes(ctypes.byref(p), b) == want
        assert lib.tm_workspace_bytes(ctypes.byref(p), 0) == lib.tm_workspace_bytes(ctypes.byref(p), 4 * R)


@pytest.mark.gpu
@pytest.mark.parametrize("R,N", [(3, 20), (400, 24), (400, 3), (500, 12), (384, 32)])
def test_caller_workspace_takes_the_same_step(R, N):
    print("case mixed workspace", R, N, flush=True)
    sys.stdout.flush()
    w = synth.make_custom(S=2, R=R, I=5, N=N)
    wd = w.to("cuda")
    f = tm.DeviceFields.of(wd)

    def step(precision, nbytes):
        ctx = tm.Context(tm.problem_of(wd, precision))
        if nbytes:
            ctx.set_workspace(nbytes(ctx))
        psi = wd.psi_n.clone()
        st, stats = ctx.newton_step(f, wd.psi_n, psi, 30, 1e-12, raise_on_status=False)
        torch.cuda.synchronize()
        ctx.close()
        assert st == tm.TM_OK
        return psi.cpu().numpy()

    own = step(tm.PREC_MIXED, None)
    np.testing.assert_array_equal(step(tm.PREC_MIXED, lambda c: c.workspace_bytes(0)), own)
    ref = step(tm.PREC_FP64, None)
    scale = np.maximum(np.max(np.abs(ref), axis=-1, keepdims=True), 1e-30)
    for b in (2 * R, 5):
        got = step(tm.PREC_MIXED, lambda c: (b + 15) * _slot(c.problem, 4))
        assert np.max(np.abs(got - ref) / scale) < 1e-8
