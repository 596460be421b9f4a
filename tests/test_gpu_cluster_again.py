"""A large scene that a workgroup gave up waiting for is solved again by one workgroup: the sums of
the stopping test are formed in the same order there, so the statistics are the same bits and the scene
stops at the same iteration, also where the tolerance is the residual of an iteration itself.

Sizes: one and two slot rows per thread, register and LDS forms, scenes of one to several
workgroups.  The wait of zero ticks gives a scene up at the first value that is not there yet.
"""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2302_14344_amd import scenes as S

pytestmark = pytest.mark.gpu

CASES = {  # scenes, subsystems, interfaces, DOF, seed
    "nc27": (3, (180, 200), (220, 230), (3, 12), 8),
    "nc51": (2, (60, 70), (190, 220), (3, 12), 2),
    "wide": (1, (12, 12), (150, 150), (3, 12), 4),
    "two-rows": (90, (60, 66), (170, 180), (3, 6), 11),
}


def _wait(pr, ticks):
    from paper_2302_14344_amd import _lib as L
    fn = L.lib().subadmm_large_scene_wait
    fn.argtypes, fn.restype = [C.c_void_p, C.c_longlong], C.c_int
    return fn(pr._h, ticks)


def _again(pr):
    from paper_2302_14344_amd import _lib as L
    fn = L.lib().subadmm_large_scene_again
    fn.argtypes, fn.restype = [C.c_void_p], C.c_int
    return fn(pr._h)


def _solve(pr, p, iters, tol, ticks):
    assert _wait(pr, ticks) > 0
    o = pr.solve(pr.tensor(p.A), pr.tensor(p.b), pr.tensor(p.J), pr.tensor(p.e), max_iters=iters, tol=tol)
    st = pr.stats()
    pr.check()
    return {k: o[k].cpu().numpy() for k in ("v_hat", "lam", "z", "u")}, st


def _problem(case):
    n, subs, ifs, ndof, seed = CASES[case]
    return S.random_assembled(seed, n_scenes=n, subs_per_scene=subs, ndof=ndof, n_if_per_scene=ifs,
                              kinds=(0, 1, 2, 3), eq_dim=(1, 6))


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("case", list(CASES))
def test_stops_where_it_would_have(case, dtype):
    from paper_2302_14344_amd.solver import Problem
    print(case, dtype, flush=True)
    p = _problem(case)
    pr = Problem.from_assembled(p, dtype=dtype)
    _, st = _solve(pr, p, 20, 0.0, -1)
    # the residual of the 20th iteration of each scene in turn, as the tolerance
    for tol in [0.0, *st["r_theta"][:3]]:
        a, sa = _solve(pr, p, 40, float(tol), -1)
        b, sb = _solve(pr, p, 40, float(tol), 0)
        for k in ("iters", "converged", "theta", "r_theta"):
            np.testing.assert_array_equal(sa[k], sb[k], err_msg=k)
        for k in a:
            np.testing.assert_array_equal(a[k], b[k], err_msg=k)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_scenes_given_up_are_counted(dtype):
    """A wait of zero ticks gives scenes up (which the equal results alone would not show), ordinary
    waits give none up."""
    from paper_2302_14344_amd.solver import Problem
    p = _problem("nc51")
    pr = Problem.from_assembled(p, dtype=dtype)
    _solve(pr, p, 40, 0.0, -1)
    assert _again(pr) == 0
    _solve(pr, p, 40, 0.0, 0)
    n = _again(pr)
    assert 1 <= n <= 2
    _solve(pr, p, 40, 0.0, -1)
    assert _again(pr) == n


def test_beside_a_kernel_that_holds_the_device():
    """A large scene on a second stream while a solve of ~27 ms holds most CUs: its workgroups are not
    all resident and waits of 20 ms may expire; the result is that of the scene alone."""
    from paper_2302_14344_amd.solver import Problem
    hold = S.random_assembled(5, n_scenes=240, subs_per_scene=(24, 24), ndof=(6, 12), n_if_per_scene=(75, 75),
                              kinds=(0, 1), eq_dim=(3, 3))
    p = S.random_assembled(8, n_scenes=1, subs_per_scene=(400, 400), ndof=(3, 12), n_if_per_scene=(1200, 1200),
                           kinds=(0, 1, 2, 3), eq_dim=(1, 6))
    one, two = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(one):
        ph = Problem.from_assembled(hold, dtype=torch.float32)
        ah = [ph.tensor(x) for x in (hold.A, hold.b, hold.J, hold.e)]
        ph.solve(*ah, max_iters=10, tol=0.0)
    with torch.cuda.stream(two):
        pr = Problem.from_assembled(p, dtype=torch.float32)
        assert _wait(pr, -1) > 256 - 240
        a = [pr.tensor(x) for x in (p.A, p.b, p.J, p.e)]
        alone = pr.solve(*a, max_iters=30, tol=0.0)
        alone_st = pr.stats()
    torch.cuda.synchronize()
    with torch.cuda.stream(one):
        ph.solve(*ah, max_iters=20000, tol=0.0)
    with torch.cuda.stream(two):
        both = pr.solve(*a, max_iters=30, tol=0.0)
        both_st = pr.stats()
        pr.check()
    torch.cuda.synchronize()
    np.testing.assert_array_equal(alone_st["theta"], both_st["theta"])
    for k in alone:
        np.testing.assert_array_equal(alone[k].cpu().numpy(), both[k].cpu().numpy(), err_msg=k)
