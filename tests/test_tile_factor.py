"""The FP64 block elimination on matrix-core tiles, from both ends of a ray, at the sizes where it can go wrong.

Tile remainders (N around multiples of 4, one to eight tiles, the cells past the sixteenth group that a second
owner holds), rays of 1 to 5 zones (no zone on one side of the meeting zone, both parities) and odd system
counts (a last wavefront with one system), each option that changes the blocks, plain and transposed, against
the oracle's block-Thomas solve.  Bar: 1e-11 of max|x|, the solves' FP64 bar (a column-dominant block costs
at most a few N ulp per zone).
"""
import dataclasses
import os
import sys

import numpy as np
import pytest
import torch

import oracle
import synth
from paper_1809_05608_amd import tm
from test_kernel_resources import BUILD, LLVM, _kernel_scratch

SHAPES = [dict(S=1, R=1, I=1, N=1), dict(S=1, R=3, I=2, N=2), dict(S=1, R=3, I=3, N=3), dict(S=3, R=1, I=4, N=4),
          dict(S=1, R=2, I=5, N=5), dict(S=1, R=3, I=12, N=8), dict(S=2, R=3, I=7, N=15), dict(S=1, R=5, I=6, N=16),
          dict(S=1, R=3, I=9, N=17), dict(S=1, R=7, I=33, N=20), dict(S=1, R=2, I=8, N=21), dict(S=1, R=3, I=5, N=24),
          dict(S=1, R=1, I=6, N=28), dict(S=1, R=3, I=4, N=29), dict(S=1, R=1, I=5, N=32)]
OPTIONS = ["plain", "lapse", "geometric", "diffusion", "sources", "zero_flux"]


def _case(shape, option):
    w = synth.make_custom(**shape)
    over = {}
    if option == "geometric":
        w = dataclasses.replace(w, limiter=synth.LIMITER_GEOM, outer_bc=synth.BC_GEOMETRIC)
    elif option == "diffusion":
        w = dataclasses.replace(w, terms=synth.TERM_DIFFUSION, limiter=synth.LIMITER_NONE)
    elif option == "sources":
        w = dataclasses.replace(w, terms=synth.TERM_EMABS | synth.TERM_NES)
    elif option == "zero_flux":
        w = dataclasses.replace(w, outer_bc=synth.BC_ZERO_FLUX, nes_amp=w.nes_amp * 30.0)
    elif option == "lapse":
        rc = 0.5 * (w.r_edge[:, 1:] + w.r_edge[:, :-1])
        over = dict(lapse=torch.sqrt(1.0 - 5e5 / rc).contiguous(), lapse_edge=torch.sqrt(1.0 - 5e5 / w.r_edge).contiguous())
    return w, over


@pytest.mark.gpu
@pytest.mark.parametrize("option", OPTIONS)
@pytest.mark.parametrize("shape", SHAPES)
def test_tile_elimination_matches_oracle(shape, option):
    print("case tiles", shape, option, flush=True)
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
    for transpose in (False, True):
        x = torch.full_like(psi_d, float("nan"))
        ctx.factor_solve(f, psi_d, rhs_d, x, transpose)
        torch.cuda.synchronize()
        x = x.cpu().numpy()
        for s in range(w.S):
            for r in range(w.R):
                xo = oracle.block_thomas_solve(*oracle.jacobian_blocks(syss[s][r], psi[s, r]), rhs[s, r],
                                               transpose=transpose)
                err = np.max(np.abs(x[s, r] - xo)) / np.max(np.abs(xo))
                assert err < 1e-11, (s, r, transpose, err)


def test_tile_kernels_use_no_scratch(tmp_path):
    obj = os.path.join(BUILD, "tm_factor_t.o")
    if not os.path.exists(obj) or not os.path.exists(f"{LLVM}/llvm-readelf"):
        pytest.skip("library objects or ROCm LLVM tools not present (run the build first)")
    scratch = _kernel_scratch(obj, str(tmp_path))
    assert len(scratch) == 32 and not any(scratch.values()), scratch
