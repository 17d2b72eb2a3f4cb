"""The coupled step's residual completion and the temperature update, sixteen zones to a wavefront, at the sizes
where that can go wrong: zone counts around multiples of sixteen and of a block's sixty-four (within a ray, and
over the flat zones of all rays), group counts around multiples of four, with and without pairs, against the
oracle.  Bars as for the other tests of these two: max|G| and de 1e-12, lepton number and T 1e-13.
"""
import sys

import numpy as np
import pytest
import torch

import oracle
import synth
from oracle import ye_coupled as yc
from paper_1809_05608_amd import tm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pairs", [False, True])
@pytest.mark.parametrize("R,I,N", [(1, 1, 1), (3, 2, 3), (1, 15, 4), (2, 16, 5), (1, 17, 8), (5, 13, 13), (1, 63, 16),
                                   (1, 64, 17), (2, 65, 20), (1, 81, 21), (3, 22, 24), (1, 33, 28)])
def test_residual_and_temperature_match_oracle(R, I, N, pairs):
    print("case coupled zones", R, I, N, pairs, flush=True)
    sys.stdout.flush()
    w = synth.make_custom(S=3, R=R, I=I, N=N)
    y = synth.ye_inputs(w, 0, R_full=R, pairs=pairs)
    rng = np.random.default_rng(N)
    psi = (w.psi_n.numpy() * rng.uniform(0.8, 1.2, w.psi_n.shape)).clip(0, 1)
    ye = y.ye_n.numpy() + 0.01 * rng.standard_normal(y.ye_n.shape)
    weights = (1.0, 1.0, 2.0)
    wd, yd = w.to("cuda"), y.to("cuda")
    ctx = tm.Context(tm.problem_of(wd))
    f = tm.DeviceFields.of(wd)
    psi_d, ye_d = torch.as_tensor(psi, device="cuda"), torch.as_tensor(ye, device="cuda")
    T1, de = torch.full_like(yd.ye_n, float("nan")), torch.full_like(yd.ye_n, float("nan"))
    ctx.temperature_update(f, yd, psi_d, ye_d, weights, yd.de_dT, yd.de_dye, T1, de)
    _, stats = ctx.ye_newton_step(f, yd, wd.psi_n, psi_d, ye_d, 0, 0.0, raise_on_status=False)
    torch.cuda.synchronize()
    T1, de, stats = T1.cpu().numpy(), de.cpu().numpy(), {k: v.cpu().numpy() for k, v in stats.items()}
    wn, yn = w.numpy(), y.numpy()
    sy = oracle.systems_from_workload(wn)
    for r, cs in enumerate(yc.coupled_systems(wn, yn)):
        u = yc.pack(psi[0, r], psi[1, r], ye[r])
        G = yc.residual(cs, yc.pack(wn["psi_n"][0, r], wn["psi_n"][1, r], cs.ye_n), u)
        assert abs(stats["res0_inf"][r] - np.max(np.abs(G))) <= 1e-12 * np.max(np.abs(G))
        L = yc.lepton_number(cs, u)
        assert abs(stats["lepton"][r] - L) <= 1e-13 * abs(L)
        de_o, T_o = yc.temperature_update(cs, [sy[2][r]], u, [psi[2, r]], weights, wn["temp"][r], yn["de_dT"][r],
                                          yn["de_dye"][r])
        assert np.max(np.abs(de[r] - de_o)) <= 1e-12 * np.max(np.abs(de_o))
        assert np.max(np.abs(T1[r] - T_o) / np.abs(T_o)) <= 1e-13
    ctx.close()
