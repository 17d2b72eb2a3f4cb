"""Newton updates through the list of active systems on both sides of the counts at which the kernel or the precision
changes (768 and 4096).  The systems at rest have psi = psi_n = 0 and no emission: their residual is exactly 0, so the
list holds exactly the moving ones, which have to reach the FP64 solution of the whole problem: 1e-10 of a zone's largest
occupation in FP64 (two solutions to rtol 1e-12), the mixed step's 1e-8 in mixed precision.
"""
import dataclasses
import sys

import numpy as np
import pytest
import torch

import synth
from paper_1809_05608_amd import tm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [tm.PREC_FP64, tm.PREC_MIXED])
@pytest.mark.parametrize("S,R,I,N,moving", [(1, 900, 4, 12, 768), (1, 900, 4, 12, 769), (2, 450, 3, 24, 768), (2, 450, 3, 24, 769),
                                            (3, 300, 5, 20, 899), (1, 4500, 2, 8, 4096), (1, 4500, 2, 8, 4097),
                                            (1, 4500, 2, 26, 4096), (1, 20000, 2, 3, 19999)])
@pytest.mark.parametrize("small", [False, True])
def test_list_holds_the_moving_systems(S, R, I, N, moving, precision, small):
    print("case system list", S, R, I, N, moving, precision, small, flush=True)
    sys.stdout.flush()
    w = synth.make_custom(S=S, R=R, I=I, N=N)
    pick = np.zeros(S * R, dtype=bool)
    pick[np.random.default_rng(moving).permutation(S * R)[:moving]] = True
    on = torch.as_tensor(pick.reshape(S, R, 1, 1))
    part = dataclasses.replace(w, psi_n=torch.where(on, w.psi_n, torch.zeros_like(w.psi_n)),
                               eta=torch.where(on, w.eta, torch.zeros_like(w.eta)))

    def step(wl, prec):
        wd = wl.to("cuda")
        ctx = tm.Context(tm.problem_of(wd, prec))
        if small:                                      # a third of the systems a launch
            ctx.set_workspace((S * R // 3 + 15) * I * ((N + 3) // 4 * 4) * ((N + 3) // 4 * 4 + 1) * (4 if prec else 8))
        psi = wd.psi_n.clone()
        st, stats = ctx.newton_step(tm.DeviceFields.of(wd), wd.psi_n, psi, 30, 1e-12, raise_on_status=False)
        torch.cuda.synchronize()
        ctx.close()
        assert st == tm.TM_OK
        return psi.cpu().numpy(), stats["iters"].cpu().numpy()

    got, iters = step(part, precision)
    assert np.all(iters[pick] > 0) and np.all(iters[~pick] == 0)
    at = pick.reshape(S, R)
    assert not got[~at].any()
    whole, _ = step(w, tm.PREC_FP64)
    scale = np.maximum(np.max(np.abs(whole), axis=-1, keepdims=True), 1e-30)
    assert np.max((np.abs(got - whole) / scale)[at]) < (1e-8 if precision == tm.PREC_MIXED else 1e-10)
