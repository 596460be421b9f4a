"""Block factorisation of the deformable-body path over block sizes (tile remainders, more tile
rows than a wave keeps in registers, blocks of less than two tiles), through whole steps of two
blocks against the oracle: FP64 1e-9, FP32 with the FP32 trial factor 1e-5 of the largest entry
after 30 iterations, as in the other parity tests of the path."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2302_14344_amd import scenes as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("trial", [False, True])
@pytest.mark.parametrize("nodes", [2, 3, 4, 6])
def test_block_sizes(nodes, trial):
    from paper_2302_14344_amd.solver import Problem, fem_state_tensors
    print(f"nodes {nodes} trial {trial}", flush=True)
    r32 = lambda a: np.asarray(a, np.float32).astype(np.float64)
    fs = S.fem_scene(seed=S.config_seed(3, 18), blocks=(2, 1, 1), nodes_per_block=nodes)
    rng = np.random.default_rng(10)
    fs = fs.with_state(r32(fs.pos + rng.uniform(-0.02, 0.02, fs.pos.shape) * fs.meta["h"]),
                       r32(rng.normal(0, 0.05, fs.pos.shape)))
    _, ref = O.fem_step(fs, max_iters=30, tol=0.0, n_threads=8)
    dtype = torch.float32 if trial else torch.float64
    pr = Problem.from_fem(fs, dtype=dtype)
    if trial:
        pr.set_fem_kappa_max(10 ** 9)
    pos, vel = fem_state_tensors(fs, dtype=dtype)
    vh, lam = pr.empty(pr.sizes.n_dof), pr.empty(pr.sizes.n_rows)
    pr.fem_step(pos, vel, max_iters=30, tol=0.0, warm="cold", v_hat=vh, lam=lam)
    _, f64 = pr.fem_block_precision()
    assert bool(f64.bool().any()) == (not trial)
    vf, lf = fs.gravity * fs.dt, fs.gravity * fs.density * 1e-6
    tol = 1e-5 if trial else 1e-9
    for g, r, floor in ((vh, ref.v_hat, vf), (lam, ref.lam, lf)):
        err = np.abs(g.detach().cpu().numpy().astype(np.float64) - r).max() / max(floor, np.abs(r).max())
        print(f"  {err:.2e}", flush=True)
        assert err <= tol
