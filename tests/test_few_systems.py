"""Newton updates of the systems still iterating: gathered through a list, and in FP64 where they are few.

The step is started with most systems at their solution and the rest at the old state, at counts around which the
factor launch changes (one, an odd pair, a wavefront per half system or four half systems to one, float32 or
FP64).  Systems at rest keep their bits; the others reach the solution that a step of all systems together
found: 1e-10 of a zone's largest occupation, two solutions to rtol 1e-12 with cells at rounding level.
"""
import sys

import numpy as np
import pytest
import torch

import synth
from paper_1809_05608_amd import tm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [tm.PREC_FP64, tm.PREC_MIXED])
@pytest.mark.parametrize("shape,moving", [
    (dict(S=2, R=3, I=9, N=20), 1), (dict(S=2, R=3, I=9, N=20), 5), (dict(S=3, R=171, I=4, N=5), 2),
    (dict(S=3, R=200, I=5, N=12), 512), (dict(S=3, R=200, I=5, N=12), 513), (dict(S=2, R=700, I=2, N=20), 1399),
    (dict(S=1, R=4100, I=2, N=8), 4096), (dict(S=1, R=4100, I=2, N=8), 4097), (dict(S=4, R=200, I=3, N=24), 777)])
@pytest.mark.parametrize("batch", [0, 3])
def test_moving_systems_reach_the_solution_of_the_whole(shape, moving, precision, batch):
    print("case few systems", shape, moving, precision, batch, flush=True)
    sys.stdout.flush()
    w = synth.make_custom(**shape)
    wd = w.to("cuda")
    f = tm.DeviceFields.of(wd)

    def step(psi, ws):
        ctx = tm.Context(tm.problem_of(wd, precision))
        if ws:
            ctx.set_workspace(ctx.workspace_bytes(max(1, w.S * w.R // ws)))
        st, stats = ctx.newton_step(f, wd.psi_n, psi, 30, 1e-12, raise_on_status=False)
        torch.cuda.synchronize()
        assert st == tm.TM_OK
        iters = stats["iters"].cpu().numpy().reshape(-1)
        ctx.close()
        return psi.cpu().numpy(), iters

    whole, _ = step(wd.psi_n.clone(), 0)
    pick = np.zeros(w.S * w.R, dtype=bool)
    pick[np.random.default_rng(moving).permutation(w.S * w.R)[:moving]] = True
    pick = pick.reshape(w.S, w.R)
    start = np.where(pick[:, :, None, None], w.psi_n.numpy(), whole)
    got, iters = step(torch.as_tensor(start, device="cuda").contiguous(), batch)
    rest = ~pick & (iters.reshape(w.S, w.R) == 0)
    np.testing.assert_array_equal(got[rest], whole[rest])
    scale = np.maximum(np.max(np.abs(whole), axis=-1, keepdims=True), 1e-30)
    assert np.max(np.abs(got - whole) / scale) < 1e-10
    assert np.all(iters.reshape(w.S, w.R)[pick] > 0)
