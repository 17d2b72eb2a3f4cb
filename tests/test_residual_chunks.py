"""The residual pass at the sizes where its mapping can go wrong: rays around multiples of a chunk (15 zones
behind a halo) for each of a ray's four parts, parts without zones, group counts around multiples of four up to
the largest, each set of terms and option, against the oracle's residual and conservation sums.  Bars as for the
other residual tests: 1e-11 relative, 1e-13 absolute.
"""
import dataclasses
import sys

import numpy as np
import pytest
import torch

import oracle
import synth
from paper_1809_05608_amd import tm
from test_tile_factor import _case

pytestmark = pytest.mark.gpu

SHAPES = [(1, 3, 1), (2, 2, 2), (3, 1, 3), (4, 2, 4), (5, 3, 5), (7, 1, 8), (14, 2, 9), (15, 1, 12), (16, 2, 13),
          (17, 1, 16), (31, 1, 17), (57, 1, 20), (58, 2, 21), (60, 1, 24), (61, 1, 25), (64, 1, 28), (65, 1, 29),
          (117, 1, 32), (121, 1, 20)]


@pytest.mark.parametrize("option", ["plain", "lapse", "geometric", "diffusion", "sources", "zero_flux", "emission"])
@pytest.mark.parametrize("shape", SHAPES)
def test_residual_and_sums_match_oracle(shape, option):
    print("case residual chunks", shape, option, flush=True)
    sys.stdout.flush()
    I, R, N = shape
    w, over = _case(dict(S=2, R=R, I=I, N=N), "plain" if option == "emission" else option)
    if option == "emission":
        w = dataclasses.replace(w, terms=synth.TERM_EMABS)
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
    wn = w.numpy()
    wn.update({k: v.numpy() for k, v in over.items()})
    syss = oracle.systems_from_workload(wn)
    for s in range(w.S):
        for r in range(w.R):
            Go = oracle.residual(syss[s][r], wn["psi_n"][s, r], psi[s, r])
            np.testing.assert_allclose(G[s, r], Go, rtol=1e-11, atol=1e-13)
            np.testing.assert_allclose(stats["res0_inf"][s, r], np.max(np.abs(Go)), rtol=1e-11)
            so = oracle.step_stats(syss[s][r], wn["psi_n"][s, r], psi[s, r])
            for k, o in (("n_tot", "n_tot"), ("e_tot", "e_tot"), ("lum_n", "lum_n")):
                np.testing.assert_allclose(stats[k][s, r], so[o], rtol=1e-11)
            size = abs(so["n_tot"]) + abs(so["q_n"]) + abs(so["b_n"])
            np.testing.assert_allclose(stats["budget_n"][s, r], so["budget"], rtol=1e-6, atol=1e-9 * size)
    ctx.close()
