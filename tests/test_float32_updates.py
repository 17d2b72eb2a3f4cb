"""Float32 Newton updates of the mixed step where the default solves in FP64 (4096 systems or fewer): with
TM_FACTOR_KERNEL set at tm_create the update stays in float32, and the step still reaches the oracle's answer at the
mixed step's 1e-8 bar.  Cold and hot zones, a lapse, the geometric options, occupations below the float32 range (the
power-of-two scaling of the right-hand side), the guard's re-run, and caller workspaces (bitwise).
"""
import dataclasses
import sys

import numpy as np
import pytest
import torch

import oracle
import synth
from paper_1809_05608_amd import tm
from test_gpu_parity import MIXED_BAR, oracle_newton, rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def in_float32(monkeypatch):
    monkeypatch.setenv("TM_FACTOR_KERNEL", "mfma")


def _step(w, over=None, nbytes=0):
    wd = w.to("cuda")
    f = tm.DeviceFields.of(wd, **{k: v.to("cuda") for k, v in (over or {}).items()})
    ctx = tm.Context(tm.problem_of(wd, tm.PREC_MIXED))
    if nbytes:
        ctx.set_workspace(nbytes)
    psi = wd.psi_n.clone()
    st, stats = ctx.newton_step(f, wd.psi_n, psi, 30, 1e-12, raise_on_status=False)
    torch.cuda.synchronize()
    ctx.close()
    assert st == tm.TM_OK, tm.STATUS_NAMES[st]
    return psi.cpu().numpy(), {k: v.cpu().numpy() for k, v in stats.items()}


@pytest.mark.parametrize("t_scale", [0.02, 1.0, 50.0])
def test_extreme_temperatures(t_scale):
    print("case float32 temperature", t_scale, flush=True)
    sys.stdout.flush()
    w = synth.make_custom(S=2, R=4, I=24, N=20)
    w = dataclasses.replace(w, temp=(w.temp * t_scale).contiguous(), nes_amp=(w.nes_amp * 10.0).contiguous())
    psi, stats = _step(w)
    ref, _ = oracle_newton(w, 30, 1e-12)
    assert rel_err(psi, ref) < MIXED_BAR
    assert not np.any(stats["flags"] & tm.FLAG_PIVOT_FALLBACK)


@pytest.mark.parametrize("N", [7, 20, 26])
@pytest.mark.parametrize("option", ["lapse", "geometric"])
def test_options(option, N):
    print("case float32 option", option, N, flush=True)
    sys.stdout.flush()
    w, over = synth.make_custom(S=2, R=3, I=30, N=N), {}
    if option == "lapse":
        rc = 0.5 * (w.r_edge[:, 1:] + w.r_edge[:, :-1])
        over = dict(lapse=torch.sqrt(1.0 - 5e5 / rc).contiguous(), lapse_edge=torch.sqrt(1.0 - 5e5 / w.r_edge).contiguous())
    else:
        w = dataclasses.replace(w, limiter=synth.LIMITER_GEOM, outer_bc=synth.BC_GEOMETRIC)
    psi, _ = _step(w, over)
    wn = w.numpy()
    wn.update({k: v.numpy() for k, v in over.items()})
    ref, _ = oracle.newton_batch(wn, max_iter=30, rtol=1e-12)
    assert rel_err(psi, ref) < MIXED_BAR


def test_below_the_float32_range():
    print("case float32 tiny occupations", flush=True)
    sys.stdout.flush()
    w = synth.make_custom(S=2, R=3, I=1, N=1)
    assert float(np.max(w.psi_n.numpy())) < 1e-150
    psi, _ = _step(w)
    ref, _ = oracle_newton(w, 30, 1e-12)
    assert rel_err(psi, ref) < MIXED_BAR


@pytest.mark.parametrize("N", [20, 26])
def test_all_systems_sent_on_by_the_guard(N, monkeypatch):
    print("case float32 guard", N, flush=True)
    sys.stdout.flush()
    monkeypatch.setenv("TM_GROWTH_LIMIT", "0")
    w = synth.make_custom(S=2, R=5, I=30, N=N)
    psi, stats = _step(w)
    ref, _ = oracle_newton(w, 30, 1e-12)
    assert rel_err(psi, ref) < MIXED_BAR
    assert np.all(stats["flags"] & tm.FLAG_PIVOT_FALLBACK)


def test_caller_workspaces_are_one_launch():
    print("case float32 workspace", flush=True)
    sys.stdout.flush()
    w = synth.make_custom(S=2, R=11, I=23, N=20)
    slot = 23 * 20 * 21 * 4
    whole, st0 = _step(w)
    for b in (1, 7):
        got, st = _step(w, nbytes=(b + 15) * slot)
        np.testing.assert_array_equal(got, whole)
        np.testing.assert_array_equal(st["iters"], st0["iters"])
