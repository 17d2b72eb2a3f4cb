"""The adjoint (always FP64) of a mixed-precision context of a few systems, after its float32-sized workspace has been
allocated by a step: a self-allocated workspace is sized again, and the adjoint is that of an FP64 context at the same
psi (bitwise: the same kernels).
"""
import sys

import pytest
import torch

import synth
from paper_1809_05608_amd import tm


@pytest.mark.gpu
@pytest.mark.parametrize("S,R", [(1, 1), (2, 3), (1, 14), (1, 40)])
def test_adjoint_after_a_mixed_step(S, R):
    print("case mixed adjoint", S, R, flush=True)
    sys.stdout.flush()
    wd = synth.make_custom(S=S, R=R, I=9, N=12).to("cuda")
    f = tm.DeviceFields.of(wd)
    mixed, exact = tm.Context(tm.problem_of(wd, tm.PREC_MIXED)), tm.Context(tm.problem_of(wd))
    psi = wd.psi_n.clone()
    mixed.newton_step(f, wd.psi_n, psi, 30, 1e-12)
    seed = torch.randn(psi.shape, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    out = []
    for ctx in (mixed, exact):
        mu, g = torch.empty_like(psi), torch.empty_like(psi)
        ctx.adjoint_step(f, wd.psi_n, psi, seed, mu, g)
        torch.cuda.synchronize()
        out.append((mu, g))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    again = wd.psi_n.clone()
    mixed.newton_step(f, wd.psi_n, again, 30, 1e-12)
    torch.cuda.synchronize()
    assert torch.equal(again, psi)
    mixed.close()
    exact.close()
