"""The tile kernel of the FP64 elimination (four half systems to a wavefront), which serves more than 768 systems:
one to eight tiles, rays of 1 to 5 zones, each option that changes the blocks, plain and transposed, an odd count (a
last wavefront with one system), and the growth guard of one system beside good ones, in both elimination kernels.

Sampled systems against the oracle.  Bar: 1e-11 of max|x|, the solves' FP64 bar.
"""
import dataclasses
import sys

import numpy as np
import pytest
import torch

import oracle
import synth
from paper_1809_05608_amd import tm
from test_tile_factor import OPTIONS, _case

pytestmark = pytest.mark.gpu

SHAPES = [(769, 1, 3), (770, 4, 4), (771, 2, 6), (769, 5, 8), (773, 3, 10), (769, 4, 12), (771, 3, 13), (770, 2, 16), (769, 5, 18),
          (771, 4, 20), (769, 2, 21), (773, 5, 24), (769, 3, 25), (771, 4, 28), (770, 1, 29), (769, 3, 32)]


def _inputs(shape, option):
    R, I, N = shape
    w, over = _case(dict(S=1, R=R, I=I, N=N), option)
    rng = np.random.default_rng(7)
    psi = (w.psi_n.numpy() * rng.uniform(0.6, 1.4, w.psi_n.shape)).clip(0, 1)
    return w, over, psi, rng.standard_normal(psi.shape)


def _systems(w, over):
    wn = w.numpy()
    wn.update({k: v.numpy() for k, v in over.items()})
    return oracle.systems_from_workload(wn)


@pytest.mark.parametrize("option", OPTIONS)
@pytest.mark.parametrize("shape", SHAPES)
def test_tiles_match_oracle(shape, option):
    print("case tile kernel", shape, option, flush=True)
    sys.stdout.flush()
    w, over, psi, rhs = _inputs(shape, option)
    syss = _systems(w, over)
    wd = w.to("cuda")
    f = tm.DeviceFields.of(wd, **{k: v.to("cuda") for k, v in over.items()})
    ctx = tm.Context(tm.problem_of(wd))
    psi_d, rhs_d = torch.as_tensor(psi, device="cuda"), torch.as_tensor(rhs, device="cuda")
    if option != "lapse":                              # no system is left to partial pivoting
        flags = torch.full((1, w.R), -1, dtype=torch.int32, device="cuda")
        ctx.factor_solve_noalloc(f, psi_d, rhs_d, torch.empty_like(psi_d), False, flags)
        assert not flags.any()
    for transpose in (False, True):
        x = torch.full_like(psi_d, float("nan"))
        ctx.factor_solve(f, psi_d, rhs_d, x, transpose)
        torch.cuda.synchronize()
        x = x.cpu().numpy()
        assert np.all(np.isfinite(x))
        for r in (0, 1, w.R // 2, w.R - 3, w.R - 2, w.R - 1):
            xo = oracle.block_thomas_solve(*oracle.jacobian_blocks(syss[0][r], psi[0, r]), rhs[0, r], transpose=transpose)
            err = np.max(np.abs(x[0, r] - xo)) / np.max(np.abs(xo))
            assert err < 1e-11, (r, transpose, err)
    ctx.close()


def _one_bad_pivot(R, I, N, odd_one):
    """Scattering in one system's innermost zone alone, its largest coupling 1, and there two neighbouring groups'
    remaining 2 x 2 block, all groups below eliminated, singular but for 1e-4 (by a negative absorption opacity): the
    multipliers of the rows behind it are 1e4 and more, both for the block and for its transpose, while partial
    pivoting finds the block of condition below 1e4.  Every other block is diagonal."""
    w = synth.make_custom(S=1, R=R, I=I, N=N, terms=synth.TERM_EMABS | synth.TERM_NES)
    rng = np.random.default_rng(7)
    psi = (w.psi_n.numpy() * rng.uniform(0.6, 1.4, w.psi_n.shape)).clip(0, 1)
    amp = torch.zeros_like(w.nes_amp)
    amp[0, odd_one, 0] = w.nes_amp[0, odd_one, 0]

    def block(amp):
        return oracle.jacobian_blocks(_systems(dataclasses.replace(w, nes_amp=amp), {})[0][odd_one], psi[0, odd_one])[0][0]

    A = block(amp)
    amp = amp / np.abs(A - np.diag(np.diag(A))).max()
    A = block(amp)
    k = (N - 3) // 2 * 2                                  # the last pair with two rows behind it
    S = A[k:, k:] - A[k:, :k] @ np.linalg.solve(A[:k, :k], A[:k, k:])
    d = S[0, 1] * S[1, 0] / S[0, 0] * (1.0 + 1e-4) - S[1, 1]
    A[k + 1, k + 1] += d
    S[1, 1] += d
    E = np.linalg.inv(S[:2, :2])
    assert min(np.abs(S[2:, :2] @ E).max(), np.abs(E @ S[:2, 2:]).max()) > 1e4 and np.linalg.cond(A) < 1e4
    ka = w.kappa_a.clone()
    ka[0, odd_one, 0, k + 1] += d / w.c_dt
    return dataclasses.replace(w, nes_amp=amp.contiguous(), kappa_a=ka.contiguous()), psi, rng.standard_normal(psi.shape)


@pytest.mark.parametrize("transpose", [False, True])
@pytest.mark.parametrize("R,I,N,odd_one", [(771, 4, 20, 0), (771, 4, 20, 1), (771, 5, 13, 770), (773, 3, 24, 400), (9, 4, 20, 3),
                                           (9, 5, 27, 8)])
def test_guard_of_one_system(R, I, N, odd_one, transpose):
    """One system trips the guard: it alone is flagged and solved by partial pivoting (bar 1e-9: its condition of 1e4
    times 20 rows of a few ulp), the others, its wavefront's other system among them, by diagonal pivots."""
    print("case guard", R, I, N, odd_one, transpose, flush=True)
    sys.stdout.flush()
    w, psi, rhs = _one_bad_pivot(R, I, N, odd_one)
    syss = _systems(w, {})
    wd = w.to("cuda")
    f = tm.DeviceFields.of(wd)
    ctx = tm.Context(tm.problem_of(wd))
    psi_d, rhs_d = torch.as_tensor(psi, device="cuda"), torch.as_tensor(rhs, device="cuda")
    x, xn = torch.full_like(psi_d, float("nan")), torch.full_like(psi_d, float("nan"))
    flags = torch.full((1, R), -1, dtype=torch.int32, device="cuda")
    ctx.factor_solve(f, psi_d, rhs_d, x, transpose)
    ctx.factor_solve_noalloc(f, psi_d, rhs_d, xn, transpose, flags)
    torch.cuda.synchronize()
    assert torch.equal(x, xn)
    want = np.zeros(R, dtype=np.int32)
    want[odd_one] = tm.FLAG_PIVOT_FALLBACK
    np.testing.assert_array_equal(flags.cpu().numpy()[0], want)
    x = x.cpu().numpy()
    for r in {odd_one, max(odd_one - 1, 0), min(odd_one + 1, R - 1), 0, R - 1}:
        xo = oracle.block_thomas_solve(*oracle.jacobian_blocks(syss[0][r], psi[0, r]), rhs[0, r], transpose=transpose)
        err = np.max(np.abs(x[0, r] - xo)) / np.max(np.abs(xo))
        assert err < (1e-9 if r == odd_one else 1e-11), (r, err)
    ctx.close()


@pytest.mark.parametrize("amplitude", [100.0, 1000.0])
@pytest.mark.parametrize("R,N", [(9, 13), (771, 13), (9, 20), (771, 20), (771, 16)])
def test_transposed_solve_under_strong_scattering_keeps_diagonal_pivots(R, N, amplitude):
    """The guard watches the Jacobian's columns, which dominate, in either direction: at 100 times the synthetic
    amplitude no system is left to partial pivoting, at 1000 times none of the transposed solve that is not of the
    plain one.  Bar: the residual of each row to 1e-12 of the sum of its terms' magnitudes (diagonal pivots without
    growth: N and the zones before, a few ulp each)."""
    print("case strong scattering", R, N, amplitude, flush=True)
    sys.stdout.flush()
    w, _, psi, rhs = _inputs((R, 6, N), "plain")
    w = dataclasses.replace(w, nes_amp=(w.nes_amp * amplitude).contiguous())
    syss = _systems(w, {})
    wd = w.to("cuda")
    f = tm.DeviceFields.of(wd)
    ctx = tm.Context(tm.problem_of(wd))
    psi_d, rhs_d = torch.as_tensor(psi, device="cuda"), torch.as_tensor(rhs, device="cuda")
    flags = {}
    for transpose in (False, True):
        x = torch.full_like(psi_d, float("nan"))
        fl = torch.full((1, R), -1, dtype=torch.int32, device="cuda")
        ctx.factor_solve_noalloc(f, psi_d, rhs_d, x, transpose, fl)
        torch.cuda.synchronize()
        flags[transpose], x = fl.cpu().numpy()[0], x.cpu().numpy()
        for r in (0, R // 2, R - 1):
            J = oracle.dense_jacobian(syss[0][r], psi[0, r])
            J = J.T if transpose else J
            v, b = x[0, r].ravel(), rhs[0, r].ravel()
            assert np.max(np.abs(J @ v - b) / (np.abs(J) @ np.abs(v) + np.abs(b))) < 1e-12, (r, transpose)
    if amplitude == 100.0:
        assert not flags[False].any() and not flags[True].any()
    assert np.sum(flags[True] != 0) <= np.sum(flags[False] != 0) + R // 100
    ctx.close()


@pytest.mark.parametrize("R,N", [(771, 20), (769, 5), (10, 20)])
def test_newton_updates_all_sent_on(R, N, monkeypatch):
    """A growth limit of 0: every system of an odd count is redone with partial pivoting, flagged, and reaches the
    oracle's solution."""
    print("case guard of all", R, N, flush=True)
    sys.stdout.flush()
    monkeypatch.setenv("TM_GROWTH_LIMIT", "0")
    w = synth.make_custom(S=1, R=R, I=4, N=N)
    wd = w.to("cuda")
    ctx = tm.Context(tm.problem_of(wd))
    psi = wd.psi_n.clone()
    st, stats = ctx.newton_step(tm.DeviceFields.of(wd), wd.psi_n, psi, 30, 1e-12, raise_on_status=False)
    torch.cuda.synchronize()
    assert st == tm.TM_OK and torch.all(stats["flags"] == tm.FLAG_PIVOT_FALLBACK)
    syss = oracle.systems_from_workload(w.numpy())
    for r in (0, 1, R - 2, R - 1):
        ref = oracle.newton(syss[0][r], w.numpy()["psi_n"][0, r], max_iter=30, rtol=1e-12).psi
        got = psi[0, r].cpu().numpy()
        assert np.max(np.abs(got - ref) / np.maximum(np.max(np.abs(ref), axis=-1, keepdims=True), 1e-30)) < 1e-10
    ctx.close()
