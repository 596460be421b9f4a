"""Large scenes cut into several workgroups that exchange shared rows in one launch, against
the phase form of the large-scene path (one launch per phase of each iteration), which does
the same arithmetic in the same order per row and interface: v_hat, lambda, z, u equal bit for
bit and the same iteration counts.

Sizes: operator rows of at most 27, 51, 75 and more columns (the register and LDS forms),
more than 512 slot rows per workgroup, single scenes and batches, every interface kind.  The
fallback for a workgroup that never sees its neighbours is forced with a wait of zero ticks.
"""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2302_14344_amd import scenes as S

pytestmark = pytest.mark.gpu

KEYS = ("v_hat", "lam", "z", "u")


def _np(t):
    return t.detach().cpu().numpy().astype(np.float64)


def _wait(pr, ticks):
    from paper_2302_14344_amd import _lib as L
    fn = L.lib().subadmm_large_scene_wait
    fn.argtypes, fn.restype = [C.c_void_p, C.c_longlong], C.c_int
    return fn(pr._h, ticks)


def _solve(pr, p, iters, tol):
    o = pr.solve(pr.tensor(p.A), pr.tensor(p.b), pr.tensor(p.J), pr.tensor(p.e), max_iters=iters, tol=tol)
    st = pr.stats()
    pr.check()
    return {k: _np(o[k]) for k in KEYS}, st


def _problem(case):
    """Random problems by their longest operator row (columns)."""
    n_scenes, subs, ifs, dim, seed, lo, hi = {
        "nc27": (3, (180, 200), (220, 230), (1, 6), 8, 20, 27), "nc51": (2, (60, 70), (190, 220), (1, 6), 2, 28, 51),
        "nc75": (2, (40, 44), (260, 290), (1, 6), 3, 52, 75), "wide": (1, (12, 12), (150, 150), (1, 6), 4, 76, 1024)}[case]
    p = S.random_assembled(seed, n_scenes=n_scenes, subs_per_scene=subs, ndof=(3, 12), n_if_per_scene=ifs,
                           kinds=(0, 1, 2, 3), eq_dim=dim)
    assert lo <= S.slot_counts(p.sub_ndof, p.if_dim, p.if_nsub, p.if_sub).max() <= hi
    return p


@pytest.mark.parametrize("tol", [0.0, 1e-4])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("case", ["nc27", "nc51", "nc75", "wide"])
def test_equal_to_the_phase_form(case, dtype, tol):
    from paper_2302_14344_amd.solver import Problem
    p = _problem(case)
    print(case, dtype, tol, flush=True)
    pr = Problem.from_assembled(p, dtype=dtype)
    assert _wait(pr, -1) > p.sub_scene[-1] + 1
    a, sa = _solve(pr, p, 60, tol)
    pr.set_large_path("phases")
    b, sb = _solve(pr, p, 60, tol)
    np.testing.assert_array_equal(sa["iters"], sb["iters"])
    np.testing.assert_array_equal(sa["converged"], sb["converged"])
    np.testing.assert_allclose(sa["r_theta"], sb["r_theta"], rtol=1e-12)
    np.testing.assert_array_equal(sb["iters_total"], 2 * sa["iters_total"])
    for k in KEYS:
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_more_than_512_rows_per_workgroup(dtype):
    """More scenes than half the workgroups: most have one each, with two slot rows per thread
    and no exchange."""
    from paper_2302_14344_amd.solver import Problem
    p = S.random_assembled(11, n_scenes=130, subs_per_scene=(60, 66), ndof=(3, 6), n_if_per_scene=(170, 180),
                           kinds=(0, 1, 2, 3), eq_dim=(1, 6))
    pr = Problem.from_assembled(p, dtype=dtype)
    assert pr.sizes.max_slot_scene > 512 and 130 <= _wait(pr, -1) <= 256
    a, sa = _solve(pr, p, 30, 1e-4)
    pr.set_large_path("phases")
    b, sb = _solve(pr, p, 30, 1e-4)
    np.testing.assert_array_equal(sa["iters"], sb["iters"])
    for k in KEYS:
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_scene_given_up_by_a_wait_is_run_again(dtype):
    """A wait of zero ticks: workgroups that do not find a neighbour's value at the first look
    leave, and the tail kernel solves the scene from its start values; statistics count it once,
    and the next launch with ordinary waits is unaffected."""
    from paper_2302_14344_amd.solver import Problem
    p = _problem("nc51")
    pr = Problem.from_assembled(p, dtype=dtype)
    pr.set_large_path("phases")
    ref, sr = _solve(pr, p, 40, 1e-5)
    pr.set_large_path(False)
    pr.reset_totals()
    for n, ticks in enumerate((0, -1, 0)):
        assert _wait(pr, ticks) > 0
        a, sa = _solve(pr, p, 40, 1e-5)
        np.testing.assert_array_equal(sa["iters"], sr["iters"])
        np.testing.assert_array_equal(sa["iters_total"], (n + 1) * sr["iters"])
        for k in KEYS:
            np.testing.assert_array_equal(a[k], ref[k], err_msg=k)


def test_two_streams_at_once():
    """Two coupled scenes stepping on two streams side by side end where each ends alone."""
    from paper_2302_14344_amd.solver import Problem, rigid_state_tensors
    sc = S.cable_scene(n_segments=160)
    alone, both = [], []
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]

    def make():
        pr = Problem.from_rigid(sc, dtype=torch.float32)
        assert _wait(pr, -1) > 1
        return pr, rigid_state_tensors(sc, dtype=torch.float32)

    pr, st = make()
    for _ in range(20):
        pr.rigid_step(*st, max_iters=30, tol=0.0, warm="prev")
    pr.check()
    alone = [_np(t) for t in st]
    pairs = []
    for s in streams:
        with torch.cuda.stream(s):
            pairs.append(make())
    torch.cuda.synchronize()
    for _ in range(20):
        for s, (pr, st) in zip(streams, pairs):
            with torch.cuda.stream(s):
                pr.rigid_step(*st, max_iters=30, tol=0.0, warm="prev")
    torch.cuda.synchronize()
    for pr, st in pairs:
        pr.check()
        both.append([_np(t) for t in st])
    for b in both:
        for x, y in zip(alone, b):
            np.testing.assert_array_equal(x, y)
