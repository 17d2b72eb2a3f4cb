"""Pair processes where a rounding or a limit shows: a neutrinosphere radius equal to a zone centre, where the limb
cosine of eq. d22 is exactly 0 and the root of 1 - (R_nu/R)^2 turns an ulp of the quotient into 1e-8, and zones at
T = 0, where every detailed-balance factor is 0.

Bars: 1e-13 of the sum of a zone's pair terms (about 50 roundings, with up to 5 ulp of the cosines at the next zone);
the coupled step's 1e-12 otherwise.
"""
import ctypes
import dataclasses
import sys

import numpy as np
import pytest
import torch

import oracle
import synth
from oracle import ye_coupled as yc
from paper_1809_05608_amd import tm
from test_gpu_pair import BAR, _compare, _oracle

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


@pytest.mark.parametrize("N", [4, 20])
def test_zones_at_zero_temperature(N):
    """As temperatures of 1e-30 MeV, which the oracle takes."""
    print("case pair zero temperature", N, flush=True)
    sys.stdout.flush()
    w = synth.make_custom(S=3, R=3, I=24, N=N)
    T = w.temp.clone()
    T[:, ::5] = 0.0
    T[2] = 0.0
    w = dataclasses.replace(w, temp=T.contiguous())
    near = dataclasses.replace(w, temp=torch.where(T == 0.0, torch.full_like(T, 1e-30), T).contiguous())
    y = dataclasses.replace(synth.ye_inputs(w, 0, R_full=3, pairs=True), pair_amp=torch.full_like(w.temp, 1e-7))
    rng = np.random.default_rng(3)
    psi = rng.uniform(0.0, 1.0, tuple(w.psi_n.shape))
    T1, de = _temperature(w, y, psi)                   # with scattering
    wn, yn = near.numpy(), y.numpy()
    sy = oracle.systems_from_workload(wn)
    for r, cs in enumerate(yc.coupled_systems(wn, yn)):
        de_o, T_o = yc.temperature_update(cs, [sy[2][r]], yc.pack(psi[0, r], psi[1, r], cs.ye_n), [psi[2, r]], (1.0,) * 3,
                                          wn["temp"][r], yn["de_dT"][r], yn["de_dye"][r])
        assert np.max(np.abs(de[r] - de_o)) <= 1e-12 * np.max(np.abs(de_o))
        assert np.max(np.abs(T1[r] - T_o)) <= 1e-12 * np.max(np.abs(T_o))
    terms = dict(terms=synth.TERM_DIFFUSION | synth.TERM_EMABS)    # the species residual divides by T
    w, near = dataclasses.replace(w, **terms), dataclasses.replace(near, **terms)
    wd, yd = w.to("cuda"), y.to("cuda")
    ctx = tm.Context(tm.problem_of(wd))
    p, ye = wd.psi_n.clone(), yd.ye_n.clone()
    st, stats = ctx.ye_newton_step(tm.DeviceFields.of(wd), yd, wd.psi_n, p, ye, 3, 0.0, raise_on_status=False)
    torch.cuda.synchronize()
    assert st == tm.TM_OK and np.all(stats["iters"].cpu().numpy() == 3)
    e, ey = _compare(w, p.cpu().numpy(), ye.cpu().numpy(), _oracle(near, y, 3, 0.0))
    assert e < BAR and ey < BAR
    ctx.close()


def test_pairs_without_a_temperature_are_refused():
    """Scattering off, pairs on, temp NULL: refused before any device work (the kernels read it)."""
    print("case pair without temp", flush=True)
    sys.stdout.flush()
    w = synth.make_custom(S=2, R=2, I=6, N=4, terms=synth.TERM_DIFFUSION | synth.TERM_EMABS)
    y = synth.ye_inputs(w, 0, R_full=2, pairs=True)
    wd, yd = w.to("cuda"), y.to("cuda")
    ctx = tm.Context(tm.problem_of(wd))
    inp, yin = ctx._inputs(tm.DeviceFields.of(wd)), ctx._ye_inputs(yd)
    inp.temp = None
    st = ctx.lib.tm_ye_newton_step(ctx._h, ctypes.byref(inp), ctypes.byref(yin), tm._ptr(wd.psi_n), tm._ptr(wd.psi_n.clone()),
                                   tm._ptr(yd.ye_n.clone()), 1, 0.0, None)
    assert tm.STATUS_NAMES[st] == "TM_ERR_INVALID_ARG"
    ctx.close()
