"""A subsystem with so many slot rows that J has more than 2^22 entries (510 DOF, 8,400 rows: the
device-memory class of the factorisation), against the oracle at 3 fixed iterations.  FP64: 1e-9
of the largest entry, the bound of the other assembled parity tests.
"""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2302_14344_amd import scenes as S


def many_rows(n, n_if, seed):
    """One scene: a subsystem of n DOF (condition 10) and one of 6, with n_if equalities of six
    rows on the large one, every 50th of them shared with the other."""
    rng = np.random.default_rng(seed)
    Q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    A = (Q * np.linspace(1.0, 10.0, n)) @ Q.T
    two = np.arange(n_if) % 50 == 0
    subs = np.stack([np.zeros(n_if, np.int64), np.where(two, 1, -1)], 1)
    dims, nsub = np.full(n_if, 6), np.where(two, 2, 1)
    nc = S.slot_counts(np.array([n, 6]), dims, nsub, subs)
    return S.AssembledProblem(np.array([n, 6], np.int32), np.array([0, 0], np.int32),
                              np.full(n_if, S.KIND_EQUALITY, np.int32), dims.astype(np.int32), nsub.astype(np.int32),
                              subs.astype(np.int32), np.zeros(n_if),
                              np.concatenate([A.ravel(), np.diag(rng.uniform(1, 2, 6)).ravel()]),
                              rng.standard_normal(n + 6), rng.standard_normal(int(nc[0]) * n + int(nc[1]) * 6),
                              rng.standard_normal(int(dims.sum())))


@pytest.mark.gpu
def test_more_than_four_million_entries_of_j():
    from paper_2302_14344_amd.solver import Problem
    p = many_rows(510, 1400, 3)
    nc = S.slot_counts(p.sub_ndof, p.if_dim, p.if_nsub, p.if_sub)
    assert nc[0] * 510 > 4244219  # the first entry whose row an FP32 quotient gets wrong
    print(f"  {int(nc[0])} slot rows", flush=True)
    pr = Problem.from_assembled(p, dtype=torch.float64)
    out = pr.solve(*(pr.tensor(x) for x in (p.A, p.b, p.J, p.e)), max_iters=3, tol=0.0)
    pr.check()
    ref = O.solve(p, p.A, p.b, p.J, p.e, max_iters=3, tol=0.0, n_threads=8)
    for k, r in (("v_hat", ref.v_hat), ("lam", ref.lam), ("z", ref.z), ("u", ref.u)):
        np.testing.assert_allclose(out[k].cpu().numpy(), r, rtol=0, atol=1e-9 * np.abs(r).max(), err_msg=k)
