"""Very many systems of five to eight groups on rays of few zones: the FP64 solve by rows in lanes, on both sides of every
line of its rule (16384 systems, eight groups, 8 zones, for the forward solve 16 with the lapse and 32 with the geometric
options), plain and transposed, sampled systems against the oracle, and Newton with it.  Bars as for the other
eliminations: 1e-11 of max|x|, Newton 1e-11 of a zone's largest occupation.
"""
import sys

import numpy as np
import pytest
import torch

import oracle
from paper_1809_05608_amd import tm
from test_tile_factor import _case

pytestmark = pytest.mark.gpu

SHAPES = [dict(S=1, R=16384, I=8, N=8), dict(S=1, R=16385, I=8, N=8), dict(S=1, R=16386, I=9, N=7), dict(S=1, R=16387, I=1, N=5),
          dict(S=2, R=8194, I=2, N=6), dict(S=1, R=16391, I=16, N=6), dict(S=1, R=16385, I=17, N=5),
          dict(S=1, R=16385, I=32, N=6), dict(S=1, R=16386, I=33, N=5), dict(S=1, R=16389, I=2, N=9)]


def _run(shape, option):
    w, over = _case(shape, option)
    wn = w.numpy()
    wn.update({k: v.numpy() for k, v in over.items()})
    wd = w.to("cuda")
    f = tm.DeviceFields.of(wd, **{k: v.to("cuda") for k, v in over.items()})
    picked = sorted({(0, 0), (0, 1), (0, w.R // 2), (w.S - 1, w.R - 3), (w.S - 1, w.R - 2), (w.S - 1, w.R - 1)})
    return w, wn, oracle.systems_from_workload(wn), wd, f, tm.Context(tm.problem_of(wd)), picked


@pytest.mark.parametrize("option", ["plain", "lapse", "geometric"])
@pytest.mark.parametrize("shape", SHAPES)
def test_solve_on_both_sides_of_the_rule(shape, option):
    print("case short systems", shape, option, flush=True)
    sys.stdout.flush()
    w, wn, syss, wd, f, ctx, picked = _run(shape, option)
    rng = np.random.default_rng(11)
    psi = (wn["psi_n"] * rng.uniform(0.6, 1.4, wn["psi_n"].shape)).clip(0, 1)
    rhs = rng.standard_normal(psi.shape)
    psi_d, rhs_d = torch.as_tensor(psi, device="cuda"), torch.as_tensor(rhs, device="cuda")
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


@pytest.mark.parametrize("slots", [0, 5000])
@pytest.mark.parametrize("option", ["plain", "geometric"])
def test_newton_of_short_systems(option, slots):
    """`slots`: a caller's workspace of that many systems, so the updates go in batches."""
    print("case short systems newton", option, slots, flush=True)
    sys.stdout.flush()
    w, wn, syss, wd, f, ctx, picked = _run(dict(S=2, R=8200, I=8, N=8), option)
    if slots:
        ctx.set_workspace(ctx.workspace_bytes(slots))
    psi = wd.psi_n.clone()
    _, stats = ctx.newton_step(f, wd.psi_n, psi, 30, 1e-12)
    torch.cuda.synchronize()
    psi, flags = psi.cpu().numpy(), stats["flags"].cpu().numpy().reshape(w.S, w.R)
    assert np.all(np.isfinite(psi)) and np.all((flags & 3) == 0)
    for s, r in picked:
        ref = oracle.newton(syss[s][r], wn["psi_n"][s, r], max_iter=30, rtol=1e-12).psi
        err = np.max(np.abs(psi[s, r] - ref) / np.maximum(np.max(np.abs(ref), axis=-1, keepdims=True), 1e-30))
        assert err < 1e-11, (s, r, err)
    ctx.close()
