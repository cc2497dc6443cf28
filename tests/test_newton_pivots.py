"""Pivots of the blocked Newton path (N > 64): the search takes the largest
magnitude by all its bits, a pivot below the reciprocal's range is divided by,
and in mixed mode well-conditioned systems converge on the FP32 factor.  Sizes
on both sides of each change of workgroup, panel and rows per lane.
"""
import numpy as np
import pytest

from test_newton_sizes import GAMMA, U, isomer_mechanism, systems

pytestmark = pytest.mark.gpu

BIG = np.finfo(np.float64).max


def solve(N, A, b, mode, **kw):
    """A [N, N, n] (exact in J: h gamma = 1) and b [N, n]."""
    import torch
    from paper_1605_03262_amd import Mechanism
    n = b.shape[1]
    J = np.where(np.eye(N, dtype=bool)[:, :, None], 1.0 - A, -A)
    assert np.array_equal(np.where(np.eye(N, dtype=bool)[:, :, None], 1.0 - J, -J), A)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    x, info = Mechanism(text=isomer_mechanism(N)).newton_solve(d(J.reshape(N * N, n)), d(np.full(n, 2.0)), d(b), GAMMA,
                                                               mode=mode, **kw)
    return x.cpu().numpy(), info.cpu().numpy()


@pytest.mark.parametrize("N", [65, 97, 129, 257, 513])
@pytest.mark.parametrize("mode", [0, 1])
def test_pivot_by_all_bits(N, mode):
    """Rows 0 and r hold 1 and 1 + e in column 0 and the largest double and 0 in
    column r.  With the larger pivot nothing overflows; eliminating row r with
    row 0 gives -(1 + e) times the largest double.  x_0 = 1, x_r = 1/2 up to a
    few units in the last place (each of four operations rounds once)."""
    rows = sorted({1, 31, 32, 63, 64, N // 2, N - 1})
    es = [2.0 ** -52, 2.0 ** -33, 2.0 ** -30, 2.0 ** -21, 2.0 ** -20, 2.0 ** -3]
    cases = [(r, e) for r in rows for e in es]
    A = np.repeat(np.eye(N)[:, :, None], len(cases), axis=2)
    b = np.ones((N, len(cases)))
    want = np.ones((N, len(cases)))
    for s, (r, e) in enumerate(cases):
        A[0, 0, s], A[0, r, s], A[r, 0, s], A[r, r, s] = 1.0, BIG, 1.0 + e, 0.0
        b[0, s], b[r, s] = BIG / 2, 1.0 + e
        want[r, s] = 0.5
    x, info = solve(N, A, b, mode)
    assert np.all(info == (0 if mode == 0 else -2)), info          # the largest double is inf in FP32
    assert np.max(np.abs(x - want)) <= 8 * U


@pytest.mark.parametrize("N", [65, 129, 193, 257, 385, 513])
@pytest.mark.parametrize("mode,exps", [(0, [-1021, -1023, -1024, -1025, -1030, -1050, -1070]),
                                       (1, [-125, -127, -128, -129, -135, -140])])
def test_last_pivot_below_the_reciprocals_range(N, mode, exps):
    """The last pivot is 2^e, where 1 / 2^e can be inf; the right-hand side there
    is 0 or 3 2^e, so every solution is exact: 0 or 3 there, 1 elsewhere.  In
    mixed mode the residual's 1 - (1 - 3 2^e) loses 3 2^e, so that only the
    systems with 0 converge on the FP32 factor."""
    cases = [(e, y) for e in exps for y in (0.0, 3.0)]
    i = N // 3
    A = np.repeat(np.eye(N)[:, :, None], len(cases), axis=2)
    b = np.ones((N, len(cases)))
    want = np.ones((N, len(cases)))
    for s, (e, y) in enumerate(cases):
        A[i, i, s] = A[N - 1, N - 1, s] = 0.0
        A[i, N - 1, s], A[N - 1, i, s] = 2.0 ** e, 1.0
        b[i, s], want[N - 1, s] = y * 2.0 ** e, y
    x, info = solve(N, A, b, mode)
    assert np.array_equal(info, [0 if mode == 0 else 1 if y == 0 else -2 for _, y in cases]), info
    assert np.array_equal(x, want)


@pytest.mark.parametrize("N", [65, 96, 97, 128, 129, 192, 193, 256, 257, 384, 385, 512, 513, 608])
def test_mixed_mode_converges_without_fp64(N):
    """The random systems of test_newton_sizes converge on the FP32 factor: its
    relative error is at most about kappa u32, below 1 (kappa below 1e7 here), so
    every sweep gains and 30 sweeps are ample; the error bar is the FP64 one."""
    import torch
    from oracle.newton_ref import newton_reference
    from paper_1605_03262_amd import Mechanism, NEWTON_MIXED
    n = 3
    J, h, b = systems(N, n)
    xr, kappa = newton_reference(J, h, GAMMA, b)
    assert np.all(kappa < 1e7)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    x, info = Mechanism(text=isomer_mechanism(N)).newton_solve(d(J), d(h), d(b), GAMMA, mode=NEWTON_MIXED, max_refine=30)
    x, info = x.cpu().numpy(), info.cpu().numpy()
    assert np.all(info >= 1), info
    err = np.max(np.abs(x - xr), axis=0) / np.max(np.abs(xr), axis=0)
    assert np.all(err <= 100 * kappa * U), err / (kappa * U)


@pytest.mark.parametrize("N", [65, 129, 513])
def test_mixed_mode_at_the_top_of_the_fp32_range(N):
    """Systems scaled by 1 and 2^115 (entries below 2^118, and 16 times that in
    the factor and 2^5 in the solution still below 2^128): the FP32 factor
    serves them without the FP64 re-solve."""
    rng = np.random.default_rng(N)
    B = rng.standard_normal((N, N))
    np.fill_diagonal(B, 0.0)
    b = rng.standard_normal(N)
    xr, kappa = np.linalg.solve(B, b), np.linalg.cond(B, np.inf)
    exps = [0, 115]
    x, info = solve(N, np.stack([2.0 ** e * B for e in exps], axis=-1), np.stack([2.0 ** e * b for e in exps], axis=-1), 1,
                    max_refine=30)
    assert np.all(info >= 1), info
    err = np.max(np.abs(x - xr[:, None]), axis=0) / np.max(np.abs(xr))
    assert np.all(err <= 100 * kappa * U), err / (kappa * U)
