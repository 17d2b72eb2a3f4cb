"""Pair processes where a rounding shows: a neutrinosphere radius equal to a zone centre, where the limb cosine of
eq. d22 is exactly 0 and the root of 1 - (R_nu/R)^2 turns an ulp of the quotient into 1e-8.

Bar: 1e-13 of the sum of a zone's pair terms (about 50 roundings, with up to 5 ulp of the cosines at the next zone).
"""
import dataclasses
import sys

import numpy as np
import pytest
import torch

import oracle
import synth
from oracle import ye_coupled as yc
from paper_1809_05608_amd import tm

pytestmark = pytest.mark.gpu


def _temperature(w, y, psi):
    wd, yd = w.to("cuda"), y.to("cuda")
    ctx = tm.Context(tm.problem_of(wd))
    T1, de = torch.full_like(yd.ye_n, float("nan")), torch.full_like(yd.ye_n, float("nan"))
    ctx.temperature_update(tm.DeviceFields.of(wd), yd, torch.as_tensor(psi, device="cuda"), yd.ye_n, (1.0,) * w.S, yd.de_dT,
                           yd.de_dye, T1, de)
    torch.cuda.synchronize()
    ctx.close()
    return T1.cpu().numpy(), de.cpu().numpy()


@pytest.mark.parametrize("R,I,N", [(1, 60, 20), (1, 40, 5), (1000, 60, 4)])
def test_neutrinosphere_at_a_zone_centre(R, I, N):
    print("case pair limb", R, I, N, flush=True)
    sys.stdout.flush()
    w = synth.make_custom(S=2, R=R, I=I, N=N)
    rc = (0.5 * (w.r_edge[0, 1:] + w.r_edge[0, :-1])).clone()
    r_nu = torch.stack([rc[8:8 + N], rc[I // 2:I // 2 + N]])
    r_nu[1, N - 1] = float("inf")                      # within its neutrinosphere everywhere
    w = dataclasses.replace(w, terms=synth.TERM_DIFFUSION, r_nu=r_nu.contiguous())
    y = synth.ye_inputs(w, 0, R_full=R, pairs=True)
    y = dataclasses.replace(y, pair_eta1=torch.zeros_like(y.pair_eta1), pair_amp=torch.full_like(y.pair_amp, 1e-7))
    psi = np.full(tuple(w.psi_n.shape), 0.5)
    _, de = _temperature(w, y, psi)
    wn, yn = w.numpy(), y.numpy()
    eps, W = oracle.transport.group_energies(wn["e_edge"])
    for r, cs in enumerate(yc.coupled_systems(wn, yn)):
        if 2 < r < R - 1:
            continue
        qa, qp, qba, qbp = yc.pair_kernels(cs)
        chi = yc.pair_chi(cs)
        size = np.einsum("ikl,k->i", 0.25 * (qp + qa * chi), eps * W)
        size = size + np.einsum("ikl,k->i", 0.25 * (qbp + qba * np.transpose(chi, (0, 2, 1))), eps * W)
        scale = yc.FOUR_PI_HC3 * yc.M_B_G / cs.rho * cs.nue.c_dt * size
        de_o, _ = yc.temperature_update(cs, [], yc.pack(psi[0, r], psi[1, r], cs.ye_n), [], (1.0, 1.0), wn["temp"][r],
                                        yn["de_dT"][r], yn["de_dye"][r])
        assert np.max(np.abs(de[r] - de_o) / scale) < 1e-13, r
