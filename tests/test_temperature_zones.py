"""The temperature update's two layouts (a thread per zone, sixteen zones to a wavefront) on both sides of the rule
between them: one to six groups, with and without pairs, the last block of zones partly filled, sampled rays against
the oracle.  Bars as for the other tests of the update: de 1e-12 of its largest, T 1e-13.
"""
import dataclasses
import os
import sys

import numpy as np
import pytest
import torch

import oracle
import synth
from oracle import ye_coupled as yc
from paper_1809_05608_amd import tm
from test_kernel_resources import BUILD, LLVM, _kernel_scratch

BASE = 4                                                # distinct rays; the others repeat them


@pytest.mark.gpu
@pytest.mark.parametrize("pairs", [False, True])
@pytest.mark.parametrize("N,zones", [(1, 51200), (2, 51200), (3, 51200), (4, 102400), (4, 819200), (5, 102400),
                                     (5, 819200), (6, 819200)])
def test_temperature_on_both_sides_of_the_rule(N, zones, pairs):
    I = 40
    w = synth.make_custom(S=3, R=BASE, I=I, N=N)
    y = synth.ye_inputs(w, 0, R_full=BASE, pairs=pairs)
    rng = np.random.default_rng(N)
    psi = (w.psi_n.numpy() * rng.uniform(0.8, 1.2, w.psi_n.shape)).clip(0, 1)
    ye = y.ye_n.numpy() + 0.01 * rng.standard_normal(y.ye_n.shape)
    weights = (1.0, 1.0, 2.0)
    wn, yn = w.numpy(), y.numpy()
    sy = oracle.systems_from_workload(wn)
    ref = []
    for r, cs in enumerate(yc.coupled_systems(wn, yn)):
        ref.append(yc.temperature_update(cs, [sy[2][r]], yc.pack(psi[0, r], psi[1, r], ye[r]), [psi[2, r]], weights,
                                         wn["temp"][r], yn["de_dT"][r], yn["de_dye"][r]))
    for R in (zones // I - 1, zones // I + 1):
        print("case temperature zones", N, R, pairs, flush=True)
        sys.stdout.flush()
        at = torch.arange(R, device="cuda") % BASE
        ray = lambda t, dim: t.to("cuda").index_select(dim, at).contiguous()
        f = tm.DeviceFields(**{k: ray(getattr(w, k), 1) for k in ("kappa_a", "eta", "kappa_s", "nes_amp")},
                            **{k: ray(getattr(w, k), 0) for k in ("r_edge", "temp")},
                            **{k: getattr(w, k).to("cuda") for k in ("e_edge", "nes_g", "r_nu")})
        yd = dataclasses.replace(y, **{k: ray(getattr(y, k), 0) for k in ("rho", "ye_n", "de_dT", "de_dye")},
                                 dka_dye=ray(y.dka_dye, 1), deta_dye=ray(y.deta_dye, 1))
        if pairs:
            yd = dataclasses.replace(yd, pair_amp=ray(y.pair_amp, 0), pair_g=y.pair_g.to("cuda"), pair_eta1=ray(y.pair_eta1, 1))
        ctx = tm.Context(tm.make_problem(3, R, I, N, w.c_dt))
        T1, de = torch.full_like(yd.ye_n, float("nan")), torch.full_like(yd.ye_n, float("nan"))
        ctx.temperature_update(f, yd, ray(torch.as_tensor(psi), 1), ray(torch.as_tensor(ye), 0), weights, yd.de_dT, yd.de_dye,
                               T1, de)
        torch.cuda.synchronize()
        ctx.close()
        assert torch.isfinite(T1).all() and torch.equal(T1[:R - BASE], T1[BASE:]) and torch.equal(de[:R - BASE], de[BASE:])
        for r in (*range(BASE), R - 1):
            de_o, T_o = ref[r % BASE]
            assert np.max(np.abs(de[r].cpu().numpy() - de_o)) <= 1e-12 * np.max(np.abs(de_o))
            assert np.max(np.abs(T1[r].cpu().numpy() - T_o) / np.abs(T_o)) <= 1e-13


def test_temperature_kernels_use_no_scratch(tmp_path):
    obj = os.path.join(BUILD, "tm_ye.o")
    if not os.path.exists(obj) or not os.path.exists(f"{LLVM}/llvm-readelf"):
        pytest.skip("library objects or ROCm LLVM tools not present (run the build first)")
    scratch = {k: v for k, v in _kernel_scratch(obj, str(tmp_path)).items() if "k_ye_temperature" in k}
    assert len(scratch) == 24 and not any(scratch.values()), scratch
