"""The deformable-body iteration tests the residual two iterations late and returns the values
of the iteration that met it: first iterations against the oracle, and a step stopped by its
tolerance against one stopped by its limit.

* FP64, 1 to 6 iterations from a warm start: 1e-9 of the largest entry (v_hat, lambda, z, u), as in
  the other parity tests of the path.
* Stopped at an iteration by the tolerance: the same bits as a step limited to that many
  iterations (the same arithmetic in the same order).
"""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2302_14344_amd import scenes as S

pytestmark = pytest.mark.gpu

CASES = {
    "2x2x2": dict(blocks=(2, 2, 2), nodes_per_block=5),
    "two-bodies": dict(blocks=(2, 1, 1), nodes_per_block=4, n_bodies=2),
}


def _np(t):
    return t.detach().cpu().numpy().astype(np.float64)


def _solver():
    from paper_2302_14344_amd.solver import Problem, fem_state_tensors
    return Problem, fem_state_tensors


def _perturbed(fs, seed, amp=0.02):
    """A deformed, moving state, rounded to FP32 (so that both types start from the same)."""
    rng = np.random.default_rng(seed)
    r = lambda a: np.asarray(a, np.float32).astype(np.float64)
    return fs.with_state(r(fs.pos + rng.uniform(-amp, amp, fs.pos.shape) * fs.meta["h"]),
                         r(rng.normal(0, 0.05, fs.pos.shape)))


def _scene_floor(fs):
    return fs.gravity * fs.dt, fs.gravity * fs.density * 1e-6


@pytest.mark.parametrize("iters", [1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("case", list(CASES))
def test_first_iterations(case, iters):
    print(f"case {case} iterations {iters}", flush=True)
    Problem, fst = _solver()
    fs = _perturbed(S.fem_scene(seed=S.config_seed(3, 16), **CASES[case]), 8)
    (p1, v1), r0 = O.fem_step(fs, max_iters=50, tol=0.0, n_threads=8)
    fs1 = fs.with_state(p1, v1)
    _, ref = O.fem_step(fs1, max_iters=iters, tol=0.0, z0=r0.z, u0=r0.u, n_threads=8)
    pr = Problem.from_fem(fs, dtype=torch.float64)
    pos, vel = fst(fs1, dtype=torch.float64)
    pr.set_warm(pr.tensor(r0.z), pr.tensor(r0.u))
    vh, lam = pr.empty(pr.sizes.n_dof), pr.empty(pr.sizes.n_rows)
    pr.fem_step(pos, vel, max_iters=iters, tol=0.0, warm="prev", v_hat=vh, lam=lam)
    assert (pr.stats()["iters"] == iters).all()
    vf, lf = _scene_floor(fs)
    z, u = pr.get_warm()
    for g, r, floor in ((vh, ref.v_hat, vf), (lam, ref.lam, lf), (z, ref.z, vf), (u, ref.u, lf)):
        np.testing.assert_allclose(_np(g), r, atol=1e-9 * max(floor, np.abs(r).max()))


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("iters", [1, 2, 3, 7, 40])
def test_stopped_by_tolerance_equals_limited(iters, dtype):
    print(f"{dtype} iterations {iters}", flush=True)
    Problem, fst = _solver()
    fs = _perturbed(S.fem_scene(seed=S.config_seed(3, 17), **CASES["2x2x2"]), 9)

    def run(limit, tol):
        pr = Problem.from_fem(fs, dtype=dtype)
        pos, vel = fst(fs, dtype=dtype)
        vh, lam = pr.empty(pr.sizes.n_dof), pr.empty(pr.sizes.n_rows)
        pr.fem_step(pos, vel, max_iters=limit, tol=tol, warm="cold", v_hat=vh, lam=lam)
        st = pr.stats()
        return [_np(x) for x in (vh, lam, pos, vel, *pr.get_warm())], st

    _, st = run(iters, 0.0)
    tol = float(st["r_theta"][0]) * (1 + 1e-9)  # met at `iters` at the latest
    got, st = run(1000, tol)
    n = int(st["iters"][0])
    assert st["converged"].all() and n <= iters
    ref, _ = run(n, 0.0)
    for a, b in zip(got, ref):
        np.testing.assert_array_equal(a, b)
