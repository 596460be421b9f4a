"""Forms of the deformable-body iteration that keep the ring of the last iterations in device memory
because it leaves too little LDS for all blocks to be resident, against the forms with the ring in
LDS.  Every form of the operator product rounds alike, so v_hat, lambda, z, u and the iteration counts
are the same bits, from a cold and a warm start, stopped by the limit at 1, 2, 3 and 7
iterations and by the tolerance.

* FP32, operators on chip: 289 blocks of 2 x 2 x 25 nodes (up to 462 slot rows, two blocks a CU)
  against the streamed operators.
* FP64 and FP32, operators streamed: many bodies of nine such blocks in one launch, more blocks than the
  device holds with the ring in LDS, against the two halves of them in a launch each.
"""
import numpy as np
import pytest
import torch

from paper_2302_14344_amd import scenes as S

pytestmark = pytest.mark.gpu


def _np(t):
    return t.detach().cpu().numpy().astype(np.float64)


def _moving(fs, seed, amp=0.02):
    rng = np.random.default_rng(seed)
    r = lambda a: np.asarray(a, np.float32).astype(np.float64)
    return fs.with_state(r(fs.pos + rng.uniform(-amp, amp, fs.pos.shape) * fs.meta["h"]),
                         r(rng.normal(0, 0.05, fs.pos.shape)))


def _bodies(fs, a, b):
    """Bodies a..b-1 of fs alone (blocks, nodes, tetrahedra and interfaces are in body order)."""
    import dataclasses
    s0, s1 = np.searchsorted(fs.sub_scene, [a, b])
    off = np.concatenate([[0], np.cumsum(fs.sub_nodes)])
    n0, n1 = off[s0], off[s1]
    t = (fs.tet_sub >= s0) & (fs.tet_sub < s1)
    j = (fs.if_sub[:, 0] >= s0) & (fs.if_sub[:, 0] < s1)
    low = lambda x, d: np.where(x >= 0, x - d, -1).astype(np.int32)
    return dataclasses.replace(
        fs, n_scenes=b - a, sub_scene=(fs.sub_scene[s0:s1] - a).astype(np.int32), sub_nodes=fs.sub_nodes[s0:s1],
        rest=fs.rest[n0:n1], pos=fs.pos[n0:n1], vel=fs.vel[n0:n1], tets=(fs.tets[t] - n0).astype(np.int32),
        tet_sub=(fs.tet_sub[t] - s0).astype(np.int32), young=fs.young[s0:s1], poisson=fs.poisson[s0:s1],
        if_kind=fs.if_kind[j], if_dim=fs.if_dim[j], if_nsub=fs.if_nsub[j], if_sub=low(fs.if_sub[j], s0),
        if_mu=fs.if_mu[j], if_node=low(fs.if_node[j], n0))


def _run(fs, dtype, tol=None, resident=None, form=None):
    """Results of a run of steps: limits 1, 2, 3 and 7 from a cold start, one more from the values it
    left, and one stopped by its tolerance (the largest residual after 30 iterations when not given)."""
    from paper_2302_14344_amd.solver import Problem, fem_state_tensors
    pr = Problem.from_fem(fs, dtype=dtype)
    if resident is not None:
        pr.set_fem_resident(resident)
    vh, lam = pr.empty(pr.sizes.n_dof), pr.empty(pr.sizes.n_rows)
    out = []
    if tol is None:
        pr.fem_step(*fem_state_tensors(fs, dtype=dtype), max_iters=30, tol=0.0, warm="cold")
        tol = float(pr.stats()["r_theta"].max()) * (1 + 1e-9)
    for warm, limit, tol_ in [("cold", 1, 0.0), ("cold", 2, 0.0), ("cold", 3, 0.0), ("cold", 7, 0.0), ("prev", 5, 0.0),
                              ("cold", 1000, tol)]:
        pos, vel = fem_state_tensors(fs, dtype=dtype)
        pr.fem_step(pos, vel, max_iters=limit, tol=tol_, warm=warm, v_hat=vh, lam=lam)
        if form is not None:
            assert pr.fem_loop_form() == form
        st = pr.stats()
        pr.check()
        out.append(([_np(x) for x in (vh, lam, *pr.get_warm())], st["iters"], st["theta"], st["converged"]))
    assert out[-1][3].all()
    return out, tol


def test_operators_on_chip():
    fs = _moving(S.fem_scene(seed=S.config_seed(3, 21), blocks=(17, 17, 1), nodes_per_block=(2, 2, 25)), 3)
    a, tol = _run(fs, torch.float32, resident=True, form=35)
    b, _ = _run(fs, torch.float32, tol, resident=False, form=0)
    for (xa, ia, ta, ca), (xb, ib, tb, cb) in zip(a, b):
        np.testing.assert_array_equal(ia, ib)
        np.testing.assert_array_equal(ta, tb)
        for x, y in zip(xa, xb):
            np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("dtype,bodies,nodes", [(torch.float64, 58, (2, 2, 25)), (torch.float32, 114, (2, 2, 27))])
def test_operators_streamed(dtype, bodies, nodes):
    print(f"  {dtype} {9 * bodies} blocks", flush=True)
    fs = _moving(S.fem_scene(seed=S.config_seed(3, 22), blocks=(3, 3, 1), nodes_per_block=nodes, n_bodies=bodies), 4)
    whole, tol = _run(fs, dtype, form=0)
    h = bodies // 2
    first, _ = _run(_bodies(fs, 0, h), dtype, tol, form=0)
    second, _ = _run(_bodies(fs, h, bodies), dtype, tol, form=0)
    for w, a, b in zip(whole, first, second):
        for k in (1, 2, 3):
            np.testing.assert_array_equal(w[k], np.concatenate([a[k], b[k]]))
        for x, y, z in zip(w[0], a[0], b[0]):
            np.testing.assert_array_equal(x, np.concatenate([y, z]))
