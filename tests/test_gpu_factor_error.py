"""Rounding error of the per-step factorisation of large subsystems (129 to 300 DOF) against the
same elimination column by column in the same precision.

The blocked form subtracts its products one after another from the entry itself, so that the
rounding follows the remainder as it shrinks.  Added up first and subtracted at the end, their
sum stays at the size of the entry and the multipliers of 300-DOF subsystems were 1.9 times as
far from the exact ones.  Here every operation of the reference rounds once in FP32 (no fused
multiply-add, a little more rounding than the kernel's); the mean over the subsystems of
the logarithm of the error (relative, root mean square over a subsystem's 18 multipliers) may exceed
the reference's by log 1.3: with 24 subsystems and a deviation of about 0.4 each, three
standard errors of the difference.
"""
import numpy as np
import pytest
import torch

from paper_2302_14344_amd import scenes as S

N_SUB, ROWS = 24, 18


def _subsystems(n):
    """One subsystem per scene, three equalities of six rows on it, condition 10, FP32 data."""
    rng = np.random.default_rng(n)
    r32 = lambda a: np.asarray(a, np.float32).astype(np.float64)
    A = np.empty((N_SUB, n, n))
    for i in range(N_SUB):
        Q, _ = np.linalg.qr(rng.standard_normal((n, n)))
        A[i] = (Q * np.geomspace(1.0, 10.0, n)) @ Q.T
        A[i] = (A[i] + A[i].T) / 2
    return (r32(A), r32(rng.standard_normal((N_SUB, n))), r32(rng.standard_normal((N_SUB, ROWS, n))),
            r32(rng.standard_normal((N_SUB, ROWS))))


def _multipliers_exact(A, b, J, e):
    be = np.trace(A) / (J * J).sum()
    return -be * (e + J @ np.linalg.solve(A + be * J.T @ J, b))


def _multipliers_fp32(A, b, J, e):
    """Eq. 23, 15, 18 and 17 with a right-looking Cholesky factor and a forward substitution by columns."""
    f = np.float32
    n = len(b)
    be = f(np.trace(A) / (J * J).sum())
    A, b, J, e = (x.astype(f) for x in (A, b, J, e))
    P = np.zeros((n, n), f)
    for k in range(ROWS):
        P += np.outer(J[k], J[k])
    K = A + be * P
    sc = f(1) / np.sqrt(np.diag(K))
    K = K * np.outer(sc, sc)
    X = np.vstack([J, b[None]]).T * sc[:, None]
    for j in range(n):
        d = np.sqrt(K[j, j])
        K[j:, j] /= d
        K[j + 1:, j + 1:] -= np.outer(K[j + 1:, j], K[j + 1:, j])
        X[j] /= d
        X[j + 1:] -= np.outer(K[j + 1:, j], X[j])
    dd = np.zeros(ROWS, f)
    for k in range(n):
        dd += X[k, :ROWS] * X[k, ROWS]
    y = be * dd
    return -(e + y / be) * be


def _mean_log_error(lam, exact):
    d = np.asarray(lam, np.float64) - exact
    return np.log(np.sqrt((d * d).sum(1) / (exact * exact).sum(1))).mean()


@pytest.mark.gpu
@pytest.mark.parametrize("n", [129, 200, 300])
def test_fp32_factorisation_rounds_like_elimination_by_columns(n):
    from paper_2302_14344_amd.solver import Problem
    A, b, J, e = _subsystems(n)
    exact = np.array([_multipliers_exact(*x) for x in zip(A, b, J, e)])
    ref = np.array([_multipliers_fp32(*x) for x in zip(A, b, J, e)])
    n_if = 3 * N_SUB
    sub = np.stack([np.repeat(np.arange(N_SUB), 3), np.full(n_if, -1)], 1).astype(np.int32)
    p = S.AssembledProblem(np.full(N_SUB, n, np.int32), np.arange(N_SUB, dtype=np.int32),
                           np.full(n_if, S.KIND_EQUALITY, np.int32), np.full(n_if, 6, np.int32),
                           np.ones(n_if, np.int32), sub, np.zeros(n_if), A.ravel(), b.ravel(), J.ravel(), e.ravel())
    pr = Problem.from_assembled(p, dtype=torch.float32, factor_fp64=False)
    out = pr.solve(*(pr.tensor(x) for x in (p.A, p.b, p.J, p.e)), max_iters=2, tol=0.0)
    pr.check()
    got = _mean_log_error(out["lam"].cpu().numpy().reshape(N_SUB, ROWS), exact)
    want = _mean_log_error(ref, exact)
    print(f"  {n} DOF: error {np.exp(got):.2e}, by columns {np.exp(want):.2e}", flush=True)
    assert got <= want + np.log(1.3)
