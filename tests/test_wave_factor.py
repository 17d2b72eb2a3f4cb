"""The eliminations with a wavefront per half ray, at the sizes where they can go wrong.

Row-group and column remainders of the block (2 NT + 1 rows from 9 to 57 over 16 columns), rays of 1 to 6 zones
(no zone on one side of the meeting zone, both parities), and each option that changes the block, against the
oracle: two coupled updates from a perturbed guess.  Bar: 1e-12 of a zone's largest occupation, as for the other
tests of the coupled step.
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
from test_tile_factor import _case

# more than 256 rays: one wavefront per half for every option
SHAPES = [(257, 5, 6), (258, 2, 20), (1, 1, 4), (2, 2, 3), (3, 3, 5), (1, 4, 8), (2, 5, 9), (3, 6, 12), (2, 4, 15), (1, 5, 17), (5, 3, 20),
          (1, 6, 21), (2, 3, 24), (1, 5, 25), (2, 4, 28)]
OPTIONS = ["plain", "lapse", "geometric", "pairs", "diffusion", "sources"]


def _zone_err(a, ref):
    return float(np.max(np.abs(a - ref) / np.maximum(np.max(np.abs(ref), axis=-1, keepdims=True), 1e-30)))


@pytest.mark.gpu
@pytest.mark.parametrize("option", OPTIONS)
@pytest.mark.parametrize("shape", SHAPES)
def test_coupled_elimination_matches_oracle(shape, option, monkeypatch):
    print("case coupled wave", shape, option, flush=True)
    sys.stdout.flush()
    if option in ("plain", "diffusion", "sources"):
        monkeypatch.setenv("TM_PIVOT", "never")            # diagonal pivots alone: no ray is sent on
    R, I, N = shape
    w = synth.make_custom(S=2, R=R, I=I, N=N)
    if option == "geometric":
        w = dataclasses.replace(w, limiter=synth.LIMITER_GEOM, outer_bc=synth.BC_GEOMETRIC)
    elif option == "diffusion":
        w = dataclasses.replace(w, terms=synth.TERM_DIFFUSION)
    elif option == "sources":
        w = dataclasses.replace(w, terms=synth.TERM_EMABS | synth.TERM_NES)
    y = synth.ye_inputs(w, 0, R_full=R, pairs=option == "pairs")
    over = {}
    if option == "lapse":
        rc = 0.5 * (w.r_edge[:, 1:] + w.r_edge[:, :-1])
        over = dict(lapse=torch.sqrt(1.0 - 5e5 / rc).contiguous(), lapse_edge=torch.sqrt(1.0 - 5e5 / w.r_edge).contiguous())
    rng = np.random.default_rng(29)
    psi0 = (w.psi_n.numpy() * rng.uniform(0.9, 1.1, w.psi_n.shape)).clip(0, 1)
    ye0 = y.ye_n.numpy() + 0.003 * rng.standard_normal(y.ye_n.shape)
    wd, yd = w.to("cuda"), y.to("cuda")
    f = tm.DeviceFields.of(wd, **{k: v.to("cuda") for k, v in over.items()})
    ctx = tm.Context(tm.problem_of(wd))
    psi, ye = torch.as_tensor(psi0, device="cuda").contiguous(), torch.as_tensor(ye0, device="cuda").contiguous()
    st, _ = ctx.ye_newton_step(f, yd, wd.psi_n, psi, ye, 2, 0.0, raise_on_status=False)
    torch.cuda.synchronize()
    assert st == tm.TM_OK
    psi, ye = psi.cpu().numpy(), ye.cpu().numpy()
    wn = w.numpy()
    wn.update({k: v.numpy() for k, v in over.items()})
    for r, cs in enumerate(yc.coupled_systems(wn, y.numpy())):
        if 2 < r < R - 2:
            continue
        u_n = yc.pack(wn["psi_n"][0, r], wn["psi_n"][1, r], cs.ye_n)
        ref = yc.newton(cs, u_n, u0=yc.pack(psi0[0, r], psi0[1, r], ye0[r]), max_iter=2, rtol=0.0).psi
        for s in range(2):
            assert _zone_err(psi[s, r], ref[:, s * N:(s + 1) * N]) < 1e-12, (s, r)
        assert np.max(np.abs(ye[r] - ref[:, 2 * N])) < 1e-12 * np.max(np.abs(ref[:, 2 * N])), r
    ctx.close()


@pytest.mark.gpu
@pytest.mark.parametrize("option", ["plain", "lapse", "geometric"])
@pytest.mark.parametrize("shape", [dict(S=2, R=384, I=3, N=4), dict(S=1, R=769, I=1, N=5), dict(S=3, R=257, I=2, N=12),
                                   dict(S=1, R=771, I=4, N=17), dict(S=1, R=770, I=5, N=20), dict(S=1, R=773, I=3, N=29),
                                   dict(S=1, R=772, I=6, N=32),
                                   dict(S=1, R=16384, I=3, N=4), dict(S=1, R=16389, I=3, N=4), dict(S=3, R=5463, I=2, N=3)])
def test_eliminations_on_both_sides_of_the_system_count(shape, option):
    """768 systems (wavefronts per half system), and just more (four half systems to a wavefront, the last one
    partly filled), and up to four groups more than 16384 systems (lanes by rows), plain and transposed, sampled
    systems against the oracle.  Bar: 1e-11 of max|x|."""
    print("case either side", shape, option, flush=True)
    sys.stdout.flush()
    w, over = _case(shape, option)
    rng = np.random.default_rng(7)
    psi = (w.psi_n.numpy() * rng.uniform(0.6, 1.4, w.psi_n.shape)).clip(0, 1)
    rhs = rng.standard_normal(psi.shape)
    wn = w.numpy()
    wn.update({k: v.numpy() for k, v in over.items()})
    syss = oracle.systems_from_workload(wn)
    wd = w.to("cuda")
    f = tm.DeviceFields.of(wd, **{k: v.to("cuda") for k, v in over.items()})
    ctx = tm.Context(tm.problem_of(wd))
    psi_d, rhs_d = torch.as_tensor(psi, device="cuda"), torch.as_tensor(rhs, device="cuda")
    picked = sorted({(0, 0), (0, 1), (0, w.R // 2), (w.S - 1, w.R - 3), (w.S - 1, w.R - 2), (w.S - 1, w.R - 1)})
    for transpose in (False, True):
        x = torch.full_like(psi_d, float("nan"))
        ctx.factor_solve(f, psi_d, rhs_d, x, transpose)
        torch.cuda.synchronize()
        x = x.cpu().numpy()
        assert np.all(np.isfinite(x))
        for s, r in picked:
            xo = oracle.block_thomas_solve(*oracle.jacobian_blocks(syss[s][r], psi[s, r]), rhs[s, r], transpose=transpose)
            err = np.max(np.abs(x[s, r] - xo)) / np.max(np.abs(xo))
            assert err < 1e-11, (s, r, transpose, err)
    ctx.close()


def test_wave_kernels_use_no_scratch(tmp_path):
    obj = os.path.join(BUILD, "tm_factor_w.o")
    if not os.path.exists(obj) or not os.path.exists(f"{LLVM}/llvm-readelf"):
        pytest.skip("library objects or ROCm LLVM tools not present (run the build first)")
    scratch = _kernel_scratch(obj, str(tmp_path))
    assert scratch and not any(scratch.values()), scratch
