"""Up to four groups a residual pass takes a thread per cell, in chunks of 62 zones with a halo; with the geometric
options only up to 768 systems.  Zone counts around a chunk, every group count, each set of terms, both sides of
the system count, against the oracle's residual and sums.  Bars as for the other residual tests: 1e-11 relative,
1e-13 absolute.
"""
import sys

import numpy as np
import pytest
import torch

import oracle
import synth
from paper_1809_05608_amd import tm
from test_tile_factor import _case

pytestmark = pytest.mark.gpu

SHAPES = [(61, 2, 1), (62, 1, 2), (63, 2, 3), (64, 1, 4), (124, 1, 4), (125, 2, 3), (300, 1, 4), (7, 384, 4), (7, 385, 3)]


@pytest.mark.parametrize("option", ["plain", "lapse", "geometric", "diffusion", "sources", "zero_flux"])
@pytest.mark.parametrize("shape", SHAPES)
def test_residual_of_few_groups_matches_oracle(shape, option):
    print("case residual few groups", shape, option, flush=True)
    sys.stdout.flush()
    I, R, N = shape
    w, over = _case(dict(S=2, R=R, I=I, N=N), option)
    rng = np.random.default_rng(I)
    psi = (w.psi_n.numpy() * rng.uniform(0.7, 1.3, w.psi_n.shape)).clip(0, 1)
    wd = w.to("cuda")
    f = tm.DeviceFields.of(wd, **{k: v.to("cuda") for k, v in over.items()})
    ctx = tm.Context(tm.problem_of(wd))
    psi_d = torch.as_tensor(psi, device="cuda")
    G = torch.full_like(psi_d, float("nan"))
    ctx.assemble(f, wd.psi_n, psi_d, G, None)
    _, stats = ctx.newton_step(f, wd.psi_n, psi_d, 0, 0.0, raise_on_status=False)
    torch.cuda.synchronize()
    G, stats = G.cpu().numpy(), {k: v.cpu().numpy().reshape(w.S, w.R) for k, v in stats.items()}
    assert np.all(np.isfinite(G))
    wn = w.numpy()
    wn.update({k: v.numpy() for k, v in over.items()})
    syss = oracle.systems_from_workload(wn)
    for s in range(w.S):
        for r in {0, w.R // 2, w.R - 1}:
            Go = oracle.residual(syss[s][r], wn["psi_n"][s, r], psi[s, r])
            np.testing.assert_allclose(G[s, r], Go, rtol=1e-11, atol=1e-13)
            np.testing.assert_allclose(stats["res0_inf"][s, r], np.max(np.abs(Go)), rtol=1e-11)
            so = oracle.step_stats(syss[s][r], wn["psi_n"][s, r], psi[s, r])
            for k, o in (("n_tot", "n_tot"), ("e_tot", "e_tot"), ("lum_n", "lum_n")):
                np.testing.assert_allclose(stats[k][s, r], so[o], rtol=1e-11)
            size = abs(so["n_tot"]) + abs(so["q_n"]) + abs(so["b_n"])
            np.testing.assert_allclose(stats["budget_n"][s, r], so["budget"], rtol=1e-6, atol=1e-9 * size)
    ctx.close()
