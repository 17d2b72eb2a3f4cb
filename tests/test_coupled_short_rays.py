"""The coupled residual completion on rays of up to sixteen zones, where each of a block's four wavefronts takes a ray:
ray counts that are no multiple of four, zone counts on both sides of sixteen, rays at rest beside rays that go on, with
and without pairs, against the oracle.  Bars as for the other tests of the coupled step: residual norm and solution
1e-12, lepton number 1e-13, updates within one.
"""
import sys

import numpy as np
import pytest
import torch

import synth
from oracle import ye_coupled as yc
from paper_1809_05608_amd import tm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pairs", [False, True])
@pytest.mark.parametrize("R,I,N", [(1, 1, 4), (2, 16, 5), (3, 15, 8), (4, 16, 13), (5, 2, 20), (6, 17, 4), (7, 16, 24), (9, 1, 28)])
def test_coupled_step_of_short_rays_matches_oracle(R, I, N, pairs):
    print("case coupled short rays", R, I, N, pairs, flush=True)
    sys.stdout.flush()
    w = synth.make_custom(S=2, R=R, I=I, N=N)
    y = synth.ye_inputs(w, 0, R_full=R, pairs=pairs)
    wn, yn = w.numpy(), y.numpy()
    systems = yc.coupled_systems(wn, yn)
    u_n = [yc.pack(wn["psi_n"][0, r], wn["psi_n"][1, r], cs.ye_n) for r, cs in enumerate(systems)]
    ref = [yc.newton(cs, u, u0=None, max_iter=30, rtol=1e-12) for cs, u in zip(systems, u_n)]
    psi0, ye0 = wn["psi_n"].copy(), yn["ye_n"].copy()
    for r in range(1, R, 2):                                  # every second ray starts where it ends
        psi0[0, r], psi0[1, r], ye0[r] = ref[r].psi[:, :N], ref[r].psi[:, N:2 * N], ref[r].psi[:, 2 * N]
    wd, yd = w.to("cuda"), y.to("cuda")
    ctx = tm.Context(tm.problem_of(wd))
    f = tm.DeviceFields.of(wd)
    psi, ye = torch.as_tensor(psi0, device="cuda").contiguous(), torch.as_tensor(ye0, device="cuda").contiguous()
    _, first = ctx.ye_newton_step(f, yd, wd.psi_n, psi.clone(), ye.clone(), 0, 0.0, raise_on_status=False)
    st, stats = ctx.ye_newton_step(f, yd, wd.psi_n, psi, ye, 30, 1e-12, raise_on_status=False)
    torch.cuda.synchronize()
    psi, ye = psi.cpu().numpy(), ye.cpu().numpy()
    first, stats = ({k: v.cpu().numpy() for k, v in s.items()} for s in (first, stats))
    assert st == tm.TM_OK and np.all(stats["flags"] == 0)
    for r, cs in enumerate(systems):
        if r % 2 == 0:
            u0 = yc.pack(psi0[0, r], psi0[1, r], ye0[r])
            G = yc.residual(cs, u_n[r], u0)
            assert abs(first["res0_inf"][r] - np.max(np.abs(G))) <= 1e-12 * np.max(np.abs(G))
            assert abs(stats["iters"][r] - ref[r].iters) <= 1 and stats["iters"][r] >= 1
        else:
            assert stats["iters"][r] <= 1                     # the oracle takes none
        for a, o in ((psi[0, r], ref[r].psi[:, :N]), (psi[1, r], ref[r].psi[:, N:2 * N])):
            assert np.max(np.abs(a - o) / np.maximum(np.max(np.abs(o), axis=-1, keepdims=True), 1e-30)) <= 1e-12
        assert np.max(np.abs(ye[r] - ref[r].psi[:, 2 * N])) <= 1e-12 * np.max(np.abs(ref[r].psi[:, 2 * N]))
        L = yc.lepton_number(cs, ref[r].psi)
        assert abs(stats["lepton"][r] - L) <= 1e-12 * abs(L)
    ctx.close()
