"""The per-step factorisation at the edges of its 16 x 16 tiles: subsystems of 1 to 129 DOF around
multiples of 16, with right-hand-side counts on both sides of a tile, one subsystem per wave,
per workgroup and (the largest) with the working arrays in device memory; against the oracle at
30 fixed iterations.  FP64: 1e-9 of the largest entry (the bound of the other parity tests).
FP32 factorisation: the backward error of an FP32 Cholesky factor, n eps32, times the condition
number 10 of the blocks and their penalty, at most 64 * 6e-8 * 10 = 4e-5, over a few tens of
iterations; bound 1e-3.
"""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2302_14344_amd import scenes as S

pytestmark = pytest.mark.gpu


def _check(p, tol, **kw):
    from paper_2302_14344_amd.solver import Problem
    pr = Problem.from_assembled(p, **kw)
    o = pr.solve(pr.tensor(p.A), pr.tensor(p.b), pr.tensor(p.J), pr.tensor(p.e), max_iters=30, tol=0.0)
    pr.check()
    ref = O.solve(p, p.A, p.b, p.J, p.e, max_iters=30, tol=0.0, n_threads=16)
    for k, r in (("v_hat", ref.v_hat), ("lam", ref.lam), ("z", ref.z), ("u", ref.u)):
        np.testing.assert_allclose(o[k].cpu().numpy().astype(np.float64), r, atol=tol * max(1.0, np.abs(r).max()), err_msg=k)


@pytest.mark.parametrize("ifs", [1, 5, 16, 40])
@pytest.mark.parametrize("n", [1, 6, 15, 16, 17, 31, 32, 33, 47, 48, 49, 64, 65, 129])
def test_tile_edges_fp64(n, ifs):
    p = S.random_assembled(700 + n, n_scenes=4, subs_per_scene=(2, 3), ndof=(n, n), n_if_per_scene=(ifs, ifs),
                           kinds=(0, 1, 2, 3), eq_dim=(1, 6))
    _check(p, 1e-9, dtype=torch.float64)


@pytest.mark.parametrize("n", [6, 16, 17, 33, 48, 64])
def test_tile_edges_fp32_factorisation(n):
    p = S.random_assembled(800 + n, n_scenes=4, subs_per_scene=(2, 3), ndof=(n, n), n_if_per_scene=(8, 8),
                           kinds=(0, 1, 2, 3), eq_dim=(1, 6))
    _check(p, 1e-3, dtype=torch.float32, factor_fp64=False)


def test_pivot_that_is_not_positive_is_reported():
    """A block whose pivot fails inside the second tile (not on its first diagonal entries)."""
    from paper_2302_14344_amd import _lib as L
    from paper_2302_14344_amd.solver import Problem
    p = S.random_assembled(900, n_scenes=1, subs_per_scene=(2, 2), ndof=(20, 20), n_if_per_scene=(2, 2), kinds=(0,))
    A = p.A.reshape(2, 20, 20).copy()
    A[1] = np.eye(20)
    A[1, 17, 18] = A[1, 18, 17] = 3.0  # indefinite, unit diagonal
    pr = Problem.from_assembled(p, rho=1e-6, dtype=torch.float64)
    pr.solve(pr.tensor(A.ravel()), pr.tensor(p.b), pr.tensor(p.J), pr.tensor(p.e), max_iters=3, tol=0.0)
    with pytest.raises(L.SubadmmError):
        pr.check()
