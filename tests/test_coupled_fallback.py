"""The coupled elimination with diagonal pivots is the one that runs: no ray of any block shape or option is sent on
to partial pivoting under the default growth limit, and one that is sent on says so in its flags.

A guard that trips where it should not (a NaN in an instance's pair, ghost-zone or hand-over terms) shows in no
result, since partial pivoting then solves the ray.
"""
import dataclasses
import sys

import numpy as np
import pytest
import torch

import synth
from oracle import ye_coupled as yc
from paper_1809_05608_amd import tm
from test_wave_factor import OPTIONS, SHAPES, _zone_err

pytestmark = pytest.mark.gpu


def _case(shape, option):
    R, I, N = shape
    w = synth.make_custom(S=2, R=R, I=I, N=N)
    if option == "geometric":
        w = dataclasses.replace(w, limiter=synth.LIMITER_GEOM, outer_bc=synth.BC_GEOMETRIC)
    elif option == "diffusion":
        w = dataclasses.replace(w, terms=synth.TERM_DIFFUSION)
    elif option == "sources":
        w = dataclasses.replace(w, terms=synth.TERM_EMABS | synth.TERM_NES)
    over = {}
    if option == "lapse":
        rc = 0.5 * (w.r_edge[:, 1:] + w.r_edge[:, :-1])
        over = dict(lapse=torch.sqrt(1.0 - 5e5 / rc).contiguous(), lapse_edge=torch.sqrt(1.0 - 5e5 / w.r_edge).contiguous())
    y = synth.ye_inputs(w, 0, R_full=R, pairs=option == "pairs")
    rng = np.random.default_rng(29)
    psi0 = (w.psi_n.numpy() * rng.uniform(0.9, 1.1, w.psi_n.shape)).clip(0, 1)
    ye0 = y.ye_n.numpy() + 0.003 * rng.standard_normal(y.ye_n.shape)
    return w, y, over, psi0, ye0


def _step(w, y, over, psi0, ye0):
    wd, yd = w.to("cuda"), y.to("cuda")
    ctx = tm.Context(tm.problem_of(wd))
    psi, ye = torch.as_tensor(psi0, device="cuda").contiguous(), torch.as_tensor(ye0, device="cuda").contiguous()
    f = tm.DeviceFields.of(wd, **{k: v.to("cuda") for k, v in over.items()})
    st, stats = ctx.ye_newton_step(f, yd, wd.psi_n, psi, ye, 2, 0.0, raise_on_status=False)
    torch.cuda.synchronize()
    ctx.close()
    return st, psi.cpu().numpy(), ye.cpu().numpy(), stats["flags"].cpu().numpy()


@pytest.mark.parametrize("option", OPTIONS)
@pytest.mark.parametrize("shape", SHAPES)
def test_no_ray_takes_partial_pivoting(shape, option):
    print("case coupled fallback", shape, option, flush=True)
    sys.stdout.flush()
    st, _, _, flags = _step(*_case(shape, option))
    assert st == tm.TM_OK and np.all(flags == 0)


@pytest.mark.parametrize("option", ["plain", "lapse", "geometric", "pairs"])
@pytest.mark.parametrize("shape", [(3, 5, 20), (258, 2, 9)])
def test_rays_sent_on_are_flagged_and_solved(shape, option, monkeypatch):
    """A growth limit of 0: every ray is redone with partial pivoting.  Bar 1e-12, as for the diagonal pivots."""
    print("case coupled fallback forced", shape, option, flush=True)
    sys.stdout.flush()
    monkeypatch.setenv("TM_GROWTH_LIMIT", "0")
    w, y, over, psi0, ye0 = _case(shape, option)
    st, psi, ye, flags = _step(w, y, over, psi0, ye0)
    assert st == tm.TM_OK and np.all(flags == tm.FLAG_PIVOT_FALLBACK)
    wn = w.numpy()
    wn.update({k: v.numpy() for k, v in over.items()})
    N = w.N
    for r, cs in enumerate(yc.coupled_systems(wn, y.numpy())):
        if 1 < r < w.R - 1:
            continue
        u_n = yc.pack(wn["psi_n"][0, r], wn["psi_n"][1, r], cs.ye_n)
        ref = yc.newton(cs, u_n, u0=yc.pack(psi0[0, r], psi0[1, r], ye0[r]), max_iter=2, rtol=0.0).psi
        for s in range(2):
            assert _zone_err(psi[s, r], ref[:, s * N:(s + 1) * N]) < 1e-12, (s, r)
        assert np.max(np.abs(ye[r] - ref[:, 2 * N])) < 1e-12 * np.max(np.abs(ref[:, 2 * N])), r
