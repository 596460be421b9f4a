"""Performance cases: what programs built on this library have it do.

Each case is one pass through the public entry points (``Problem``, ``Mlp``) with the data a
simulation, planning or training program holds at that moment: articulated batches stepped or
rolled out from a given state, single coupled scenes at the fixed iteration counts of the
evaluation protocol, deformable bodies, assembled problems handed to ``solve``, and the
training step and inference of the warm-start networks.

``exact`` computes the same results in 64 bits with plain torch operations: the construction
of the rigid and deformable models, the ADMM iteration with explicit slot vectors, and the
networks.  It shares no code with the library.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2302_14344_amd import scenes as S
from paper_2302_14344_amd.solver import Mlp, Problem

DTYPES = {"f32": torch.float32, "f64": torch.float64}


# ---------------------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------------------
def listed():
    return [
        # one small articulated mechanism in a real-time loop: latency of a single call (the
        # small-chain workload: 8 links, 4 subsystems, FP64, uniform penalty)
        {"name": "chain_f64", "kind": "rigid", "scene": "chain", "size": 8, "dtype": "f64", "rho": 1e3,
         "iters": 200, "tol": 1e-6, "steps": 1, "form": "eager"},
        # the benchmark's batch of legged robots, one control step replayed from a graph
        {"name": "legged_1024", "kind": "rigid", "scene": "legged", "size": 1024, "dtype": "f32", "rho": 0.0,
         "iters": 1000, "tol": 1e-6, "steps": 1, "form": "graph"},
        # sampling-based planning: a batch rolled out over a short horizon in one launch (two
        # steps in FP32; drawn FP64 ones go further, where rounding stays far below the result)
        {"name": "legged_rollout_512", "kind": "rigid", "scene": "legged", "size": 512, "dtype": "f32", "rho": 0.0,
         "iters": 1000, "tol": 1e-6, "steps": 2, "form": "rollout"},
        # generic solver entry: ragged small subsystems of every interface kind, some with
        # three or four members (a caller with its own construction)
        {"name": "solve_ragged", "kind": "solve", "scenes": 200, "subs": 6, "n_lo": 4, "n_hi": 48, "ifs": 12,
         "members": 4, "dtype": "f32", "iters": 200, "tol": 1e-6},
        # the same entry with subsystems whose factorisation exceeds the LDS
        {"name": "solve_large_blocks", "kind": "solve", "scenes": 3, "subs": 4, "n_lo": 40, "n_hi": 320, "ifs": 14,
         "members": 2, "dtype": "f64", "iters": 200, "tol": 1e-6},
        # the 40^3-node deformable lattice (512 blocks), one step run to tolerance
        {"name": "fem_lattice", "kind": "fem", "bx": 8, "by": 8, "bz": 8, "q": 5, "dtype": "f32", "iters": 20000,
         "tol": 1e-6},
        # the beam of the evaluation protocol at 60 iterations
        {"name": "fem_beam", "kind": "fem", "bx": 20, "by": 1, "bz": 1, "q": 0, "dtype": "f32", "iters": 60,
         "tol": 0.0},
        # the cable of the evaluation protocol (one coupled scene of 162 subsystems), 60 iterations
        {"name": "cable_640", "kind": "rigid", "scene": "cable", "size": 640, "dtype": "f32", "rho": 0.0,
         "iters": 60, "tol": 0.0, "steps": 1, "form": "graph"},
        # the granular stirring of the evaluation protocol (217 subsystems), 60 iterations
        {"name": "stir_216", "kind": "rigid", "scene": "stir", "size": 6, "dtype": "f32", "rho": 0.0,
         "iters": 60, "tol": 0.0, "steps": 1, "form": "eager"},
        # boxes stacked around arms, 64 scenes of ~1.5k slot rows, bounded iterations
        {"name": "mixed_64", "kind": "rigid", "scene": "mixed", "size": 64, "dtype": "f32", "rho": 0.0,
         "iters": 100, "tol": 1e-6, "steps": 1, "form": "eager"},
        # one Adam step of the joint warm-start network on a training minibatch
        {"name": "mlp_train", "kind": "mlp", "n_in": 27, "n_out": 15, "width": 256, "layers": 4, "batch": 8192,
         "train": True},
        # inference of the joint network over the benchmark batch's joints
        {"name": "mlp_infer", "kind": "mlp", "n_in": 27, "n_out": 15, "width": 256, "layers": 4, "batch": 15393,
         "train": False},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    fam = rng.choice(["chain", "legged", "rollout", "solve", "solve_large", "fem", "beam", "cable", "stir", "mixed",
                      "train", "infer"])
    rigid = {"kind": "rigid", "rho": 0.0, "steps": 1}
    if fam == "chain":
        return dict(rigid, scene="chain", size=rng.randint(3, 24), dtype=rng.choice(["f64", "f32"]), rho=1e3,
                    iters=rng.randint(50, 200), tol=1e-6, form=rng.choice(["eager", "graph"]))
    if fam == "legged":
        return dict(rigid, scene="legged", size=_log(rng, 1, 1024), dtype="f32", iters=rng.randint(200, 1000),
                    tol=1e-6, form=rng.choice(["eager", "graph"]))
    if fam == "rollout":
        dt = rng.choice(["f32", "f64"])
        return dict(rigid, scene="legged", size=_log(rng, 1, 512 if dt == "f32" else 128), dtype=dt,
                    iters=rng.randint(300, 1000), tol=1e-6, steps=2 if dt == "f32" else rng.randint(2, 6),
                    form="rollout")
    if fam == "cable":
        return dict(rigid, scene="cable", size=_log(rng, 40, 2560), dtype=rng.choice(["f32", "f64"]),
                    iters=rng.randint(30, 90), tol=0.0, form=rng.choice(["eager", "graph"]))
    if fam == "stir":
        return dict(rigid, scene="stir", size=rng.randint(3, 10), dtype="f32", iters=rng.randint(30, 90), tol=0.0,
                    form=rng.choice(["eager", "graph"]))
    if fam == "mixed":
        return dict(rigid, scene="mixed", size=_log(rng, 1, 64), dtype="f32", iters=rng.randint(30, 100), tol=1e-6,
                    form=rng.choice(["eager", "graph"]))
    if fam == "solve":
        lo = rng.randint(1, 12)
        return {"kind": "solve", "scenes": _log(rng, 1, 400), "subs": rng.randint(2, 8), "n_lo": lo,
                "n_hi": rng.randint(lo + 1, 48), "ifs": rng.randint(2, 12), "members": rng.choice([2, 4]),
                "dtype": rng.choice(["f32", "f64"]), "iters": rng.randint(50, 200), "tol": 1e-6}
    if fam == "solve_large":
        return {"kind": "solve", "scenes": rng.randint(1, 4), "subs": rng.randint(2, 4), "n_lo": 40,
                "n_hi": rng.randint(100, 320), "ifs": rng.randint(4, 14), "members": 2,
                "dtype": rng.choice(["f32", "f64"]), "iters": rng.randint(50, 200), "tol": 1e-6}
    if fam == "fem":
        return {"kind": "fem", "bx": rng.randint(1, 8), "by": rng.randint(1, 8), "bz": rng.randint(1, 6),
                "q": rng.choice([3, 4, 5]), "dtype": rng.choice(["f32", "f32", "f64"]), "iters": rng.randint(60, 400),
                "tol": 1e-6}
    if fam == "beam":
        return {"kind": "fem", "bx": _log(rng, 5, 160), "by": 1, "bz": 1, "q": 0, "dtype": "f32",
                "iters": rng.randint(30, 90), "tol": 0.0}
    ci = rng.random() < 0.5
    return {"kind": "mlp", "n_in": 12 if ci else 27, "n_out": 6 if ci else 15, "width": 256, "layers": 4,
            "batch": _log(rng, 50, 8192 if fam == "train" else 16384), "train": fam == "train"}


# ---------------------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------------------
@functools.lru_cache(maxsize=8)
def _rigid_scene(scene, size):
    """Topology and model of a scene (the handle a program keeps); states come from the seed."""
    if scene == "chain":
        return S.chain_scene(S.config_seed(1), n_links=size)
    if scene == "legged":
        return S.legged_scenes(size, seed=S.config_seed(2))
    if scene == "cable":
        return S.cable_scene(n_segments=size)
    if scene == "stir":
        return S.stir_scene(n_side=size)
    return S.mixed_scenes(size)


def _rigid_state(case, seed):
    """Start-of-step state (pos, rot, vel, omega) in FP64."""
    sc = _rigid_scene(case["scene"], case["size"])
    rng = np.random.Generator(np.random.PCG64([seed, sc.n_bodies]))
    pos, rot, vel, om = sc.state()
    body_scene = sc.sub_scene[sc.body_sub]
    if case["scene"] in ("chain", "legged"):
        # touching down: the lowest contact point up to 0.5 mm above the ground, the whole
        # mechanism moving sideways and downwards
        z = pos[sc.contact_body, 2] + np.einsum("qc,qc->q", rot[sc.contact_body, 2], sc.contact_point)
        low = np.full(sc.n_scenes, np.inf)
        np.minimum.at(low, body_scene[sc.contact_body], z)
        pos[:, 2] += (rng.uniform(0.0, 5e-4, sc.n_scenes) - low)[body_scene]
        v = rng.normal(0.0, 0.2, (sc.n_scenes, 3))
        v[:, 2] = -rng.uniform(0.0, 0.5, sc.n_scenes)
        vel += v[body_scene]
        om += rng.normal(0.0, 0.05, om.shape)
    elif case["scene"] == "cable":
        vel[:-2] = rng.normal(0.0, 0.01, vel[:-2].shape)
    elif case["scene"] == "stir":
        vel += rng.normal(0.0, 5e-3, vel.shape)
    else:
        vel += rng.normal(0.0, 0.02, vel.shape)
    return sc, pos, rot, vel, om


@functools.lru_cache(maxsize=4)
def _fem_scene(bx, by, bz, q):
    if q == 0:
        return S.beam_scene(pieces=bx)
    return S.fem_scene(blocks=(bx, by, bz), nodes_per_block=q)


def _fem_state(case, seed):
    """A slightly strained, moving body about to touch the ground (coincident node copies share
    their position and velocity)."""
    fs = _fem_scene(case["bx"], case["by"], case["bz"], case["q"])
    rng = np.random.Generator(np.random.PCG64([seed, fs.n_nodes]))
    F = np.eye(3) + rng.normal(0.0, 2e-3, (3, 3))
    pos = fs.rest @ F.T
    pos[:, 2] += rng.uniform(0.0, 2e-4) - pos[:, 2].min()
    vel = pos @ rng.normal(0.0, 0.2, (3, 3)).T + [0.2, 0.0, -0.1]
    return fs, pos, vel


@functools.lru_cache(maxsize=8)
def _solve_topology(scenes, subs, n_lo, n_hi, ifs, members):
    return S.random_assembled(S.config_seed(9), n_scenes=scenes, subs_per_scene=(2, subs), ndof=(n_lo, n_hi),
                              n_if_per_scene=(2, ifs), kinds=(0, 1, 2, 3), max_members=members)


def _solve_inputs(case, seed):
    p = _solve_topology(case["scenes"], case["subs"], case["n_lo"], case["n_hi"], case["ifs"], case["members"])
    rng = np.random.Generator(np.random.PCG64([seed, p.n_sub]))
    scale = np.repeat(rng.uniform(0.5, 2.0, p.n_sub), p.sub_ndof.astype(np.int64) ** 2)
    # rows of unit length on average, whatever the subsystem's size
    nc = S.slot_counts(p.sub_ndof, p.if_dim, p.if_nsub, p.if_sub)
    rows = np.repeat(1.0 / np.sqrt(p.sub_ndof), nc * p.sub_ndof)
    return p, p.A * scale, rng.standard_normal(p.b.size), rng.standard_normal(p.J.size) * rows, rng.standard_normal(p.e.size)


def _mlp_inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    w = [case["n_in"]] + [case["width"]] * (case["layers"] - 1) + [case["n_out"]]
    params = []
    for k in range(len(w) - 1):
        params.append(torch.randn(w[k + 1] * w[k], generator=g, device="cuda") * math.sqrt(2.0 / w[k]))
        params.append(torch.randn(w[k + 1], generator=g, device="cuda") * 0.1)
    x = torch.randn(case["batch"], w[0], generator=g, device="cuda") * 2.0 + 0.5
    target = torch.randn(case["batch"], w[-1], generator=g, device="cuda")
    wt = torch.rand(case["batch"], w[-1], generator=g, device="cuda")
    scale = 0.5 + 0.1 * torch.rand(w[0], generator=g, device="cuda")
    shift = -0.25 + 0.1 * torch.rand(w[0], generator=g, device="cuda")
    return w, torch.cat(params), x, target, wt, scale, shift


def prepare(case, seed):
    if case["kind"] == "rigid":
        dt = DTYPES[case["dtype"]]
        sc, pos, rot, vel, om = _rigid_state(case, seed)
        pr = Problem.from_rigid(sc, rho=case["rho"], dtype=dt)
        start = pr.tensor(np.concatenate([a.reshape(-1) for a in (pos, rot, vel, om)]))
        flat = start.clone()
        nb = sc.n_bodies
        views = [flat[:3 * nb], flat[3 * nb:12 * nb], flat[12 * nb:15 * nb], flat[15 * nb:]]
        zero = torch.zeros(pr.sizes.n_slot, dtype=dt, device=pr.device)
        return {"case": case, "pr": pr, "start": start, "flat": flat, "views": views, "zero": zero,
                "v_hat": pr.empty(pr.sizes.n_dof), "lam": pr.empty(pr.sizes.n_rows)}
    if case["kind"] == "fem":
        fs, pos, vel = _fem_state(case, seed)
        pr = Problem.from_fem(fs, dtype=DTYPES[case["dtype"]])
        start = pr.tensor(np.concatenate([pos.reshape(-1), vel.reshape(-1)]))
        flat = start.clone()
        return {"case": case, "pr": pr, "start": start, "flat": flat, "views": list(flat.chunk(2)),
                "v_hat": pr.empty(pr.sizes.n_dof), "lam": pr.empty(pr.sizes.n_rows)}
    if case["kind"] == "solve":
        p, *arr = _solve_inputs(case, seed)
        pr = Problem.from_assembled(p, dtype=DTYPES[case["dtype"]])
        return {"case": case, "pr": pr, "args": [pr.tensor(a) for a in arr]}
    w, params, x, target, wt, scale, shift = _mlp_inputs(case, seed)
    net = Mlp(w, case["batch"])
    net.set_params(params)
    net.set_input_affine(scale, shift)
    return {"case": case, "net": net, "x": x, "target": target, "wt": wt, "step": 0}


def run(st):
    case = st["case"]
    if case["kind"] == "rigid":
        pr = st["pr"]
        st["flat"].copy_(st["start"])
        args = dict(max_iters=case["iters"], tol=case["tol"], v_hat=st["v_hat"], lam=st["lam"])
        if case["form"] == "eager":
            pr.rigid_step(*st["views"], warm="cold", **args)
        else:
            pr.set_warm(st["zero"], st["zero"])
            if case["form"] == "graph":
                pr.rigid_step(*st["views"], warm="prev", graph=True, **args)
            else:
                pr.rigid_steps(*st["views"], case["steps"], warm="prev", **args)
        return {"state": st["views"], "v_hat": st["v_hat"], "lam": st["lam"]}
    if case["kind"] == "fem":
        st["flat"].copy_(st["start"])
        st["pr"].fem_step(*st["views"], max_iters=case["iters"], tol=case["tol"], warm="cold", v_hat=st["v_hat"],
                          lam=st["lam"])
        return {"state": st["views"], "v_hat": st["v_hat"], "lam": st["lam"]}
    if case["kind"] == "solve":
        return st["pr"].solve(*st["args"], max_iters=case["iters"], tol=case["tol"], warm="cold")
    net = st["net"]
    if not case["train"]:
        return net.infer(st["x"])
    st["step"] += 1
    y = net.forward(st["x"])
    loss, grad = net.backward(st["target"], st["wt"], want_grad=True)
    net.adam(1e-3, st["step"])
    return {"y": y, "loss": loss, "grad": grad}


# ---------------------------------------------------------------------------------------
# Work of one pass
# ---------------------------------------------------------------------------------------
# x-updates counted for a run to tolerance: about what the benchmark batch, the lattice and
# random problems take per step
TOL_ITERS = {"rigid": 250, "solve": 100, "fem": 1500}


def work(case):
    """Inputs read once and outputs written once; the factorisations, and per x-update one
    multiply-add per entry of each subsystem's slot-space operator."""
    if case["kind"] == "mlp":
        w = [case["n_in"]] + [case["width"]] * (case["layers"] - 1) + [case["n_out"]]
        par = sum(a * b + b for a, b in zip(w[:-1], w[1:]))
        mac = sum(a * b for a, b in zip(w[:-1], w[1:]))
        if not case["train"]:
            return {"bytes": 4 * (par + case["batch"] * (w[0] + w[-1])), "flops": 2.0 * case["batch"] * mac}
        # parameters and both moments read and written, gradient written, activations used twice
        return {"bytes": 4 * (8 * par + case["batch"] * (w[0] + 4 * w[-1])),
                "flops": 2.0 * case["batch"] * (3 * mac - w[0] * w[1])}
    R = 8 if case["dtype"] == "f64" else 4
    iters = case["iters"] if case["tol"] == 0.0 else min(case["iters"], TOL_ITERS[case["kind"]])
    if case["kind"] == "solve":
        p = _solve_topology(case["scenes"], case["subs"], case["n_lo"], case["n_hi"], case["ifs"], case["members"])
        model = p.A.size + p.b.size + p.J.size + p.e.size
        steps = 1
    elif case["kind"] == "fem":
        p = _fem_scene(case["bx"], case["by"], case["bz"], case["q"])
        model = 2 * 3 * p.n_nodes + 2 * p.n_tets + 3 * p.n_nodes
        steps = 1
    else:
        p = _rigid_scene(case["scene"], case["size"])
        model = (18 + 4) * p.n_bodies + 18 * len(p.joint_body) + 20 * len(p.link_type) + 3 * len(p.contact_body)
        steps = case["steps"]
    n = p.sub_ndof.astype(np.float64)
    nc = S.slot_counts(p.sub_ndof, p.if_dim, p.if_nsub, p.if_sub).astype(np.float64)
    rows, slots = int(p.if_dim.sum()), int(nc.sum())
    out = int(n.sum()) + rows + (2 * slots if case["kind"] == "solve" else 2 * int(n.sum()))
    m = np.minimum(nc, n)  # constrained DOFs at most
    factor = (n ** 3 / 3 + n * n * nc if case["kind"] != "fem" else n ** 3 / 3 + m ** 3 / 3 + m ** 3 / 3).sum()
    per_iter = (m * m if case["kind"] == "fem" else nc * nc).sum()
    return {"bytes": float(R * (model + out)), "flops": float(steps * (factor + 2.0 * iters * per_iter))}


# ---------------------------------------------------------------------------------------
# The same results in 64 bits
# ---------------------------------------------------------------------------------------
def _f64(a):
    return torch.as_tensor(np.asarray(a), dtype=torch.float64, device="cuda")


def _i64(a):
    return torch.as_tensor(np.asarray(a).astype(np.int64), device="cuda")


class _Slots:
    """Slot rows: per subsystem the rows of its interfaces, by interface then row."""

    def __init__(self, p):
        ns, ni = p.n_sub, p.n_if
        width = p.if_sub.shape[1]
        ent = [(p.if_sub[j, m], j, k, m) for j in range(ni) for m in range(min(int(p.if_nsub[j]), width))
               for k in range(int(p.if_dim[j]))]
        ent = np.array(ent, np.int64).reshape(-1, 4)
        ent = ent[np.lexsort((ent[:, 2], ent[:, 1], ent[:, 0]))]
        self.n = len(ent)
        self.nc = np.bincount(ent[:, 0], minlength=ns) if self.n else np.zeros(ns, np.int64)
        first = np.concatenate([[0], np.cumsum(self.nc)])
        row0 = np.concatenate([[0], np.cumsum(p.if_dim)])
        self.start = np.zeros((ni, width), np.int64)  # first slot of each member
        sel = ent[:, 2] == 0
        self.start[ent[sel, 1], ent[sel, 3]] = np.nonzero(sel)[0]
        self.first, self.row0 = first, row0
        self.sub_np = ent[:, 0]
        self.loc_np = np.arange(self.n) - first[ent[:, 0]]
        self.sub, self.loc = _i64(self.sub_np), _i64(self.loc_np)
        self.row = _i64(row0[ent[:, 1]] + ent[:, 2])
        self.scene = _i64(p.sub_scene[ent[:, 0]])
        self.n_scene = int(p.sub_scene[-1]) + 1
        self.row_scene = _i64(np.repeat(p.sub_scene[p.if_sub[:, 0]], p.if_dim))
        self.kind = _i64(np.repeat(p.if_kind, p.if_dim))
        k = getattr(p, "if_k", None)
        al = getattr(p, "if_alpha", None)
        self.k = _f64(np.repeat(k if k is not None else np.zeros(ni), p.if_dim))
        self.alpha = _f64(np.repeat(al if al is not None else np.zeros(ni), p.if_dim))
        con = np.nonzero(np.asarray(p.if_kind) == 1)[0]
        self.con = _i64(row0[con])
        self.mu = _f64(np.asarray(p.if_mu)[con])


def _admm(sl, beta, x_of, v_of, e, iters, tol, z0=None, u0=None):
    """The iteration on explicit slot vectors; a scene stops on its own test.  beta per
    subsystem, x_of(w) = J v_hat, v_of(w) = v_hat, with w = beta z - u."""
    be = beta[sl.sub]
    z = torch.zeros(sl.n, dtype=torch.float64, device="cuda") if z0 is None else z0
    u = torch.zeros_like(z) if u0 is None else u0
    y, w = be * z + u, be * z - u
    rows = sl.row_scene.numel()
    wsum = torch.zeros(rows, dtype=torch.float64, device="cuda").index_add_(0, sl.row, 1.0 / be)
    live = torch.ones(sl.n_scene, dtype=torch.bool, device="cuda")
    kinds = [bool((sl.kind == k).any()) for k in range(4)]
    for it in range(iters):
        on = live[sl.scene]
        yn = torch.where(on, be * x_of(w) + u, y)
        th = torch.zeros(sl.n_scene, dtype=torch.float64, device="cuda").index_add_(0, sl.scene, (yn - y) ** 2)
        yy = torch.zeros(sl.n_scene, dtype=torch.float64, device="cuda").index_add_(0, sl.scene, yn * yn)
        y = yn
        live = live & (th > tol * tol * yy.clamp(min=1e-24))
        if it + 1 == iters or (it % 16 == 15 and tol > 0 and not bool(live.any())):
            break
        sy = torch.zeros(rows, dtype=torch.float64, device="cuda").index_add_(0, sl.row, y / be)
        lam = -(e + sy) / wsum
        if kinds[3]:
            lam = torch.where(sl.kind == 3, -sl.k * (e + sl.alpha * sy) / (1.0 + wsum * sl.alpha * sl.k), lam)
        if kinds[2]:
            lam = torch.where(sl.kind == 2, lam.clamp(min=0.0), lam)
        if kinds[1]:
            c = sl.con
            ln = lam[c].clamp(min=0.0)
            tn = torch.hypot(lam[c + 1], lam[c + 2])
            f = torch.where(tn > sl.mu * ln, sl.mu * ln / tn.clamp(min=1e-300), torch.ones_like(tn))
            lam = lam.index_put((c,), ln).index_put((c + 1,), f * lam[c + 1]).index_put((c + 2,), f * lam[c + 2])
        on = live[sl.scene]
        ls = lam[sl.row]
        u = torch.where(on, -ls, u)
        w = torch.where(on, y + 2.0 * ls, w)
    lam = torch.zeros(rows, dtype=torch.float64, device="cuda")
    lam[sl.row] = -u
    return v_of(w), lam, (w + u) / be, u


class _Padded:
    """Dense per-subsystem operators, zero padded to the largest subsystem."""

    def __init__(self, p, sl):
        self.sl = sl
        self.n = p.sub_ndof.astype(np.int64)
        self.nm, self.cm = int(self.n.max()), max(1, int(sl.nc.max()))
        self.n_sub = p.n_sub
        dof_sub = np.repeat(np.arange(p.n_sub), self.n)
        dof_loc = np.arange(dof_sub.size) - np.concatenate([[0], np.cumsum(self.n)])[dof_sub]
        self.dof = _i64(dof_sub * self.nm + dof_loc)
        self.slot = sl.sub * self.cm + sl.loc
        self.A = torch.zeros(p.n_sub, self.nm, self.nm, dtype=torch.float64, device="cuda")
        self.J = torch.zeros(p.n_sub, self.cm, self.nm, dtype=torch.float64, device="cuda")
        self.b = torch.zeros(p.n_sub, self.nm, dtype=torch.float64, device="cuda")

    def solve(self, e, rho, iters, tol, z0=None, u0=None):
        tr = self.A.diagonal(dim1=1, dim2=2).sum(1)
        tj = (self.J ** 2).sum((1, 2))
        beta = torch.full_like(tr, rho) if rho > 0 else torch.where(tj > 0, tr / tj.clamp(min=1e-300), torch.ones_like(tr))
        JT = self.J.transpose(1, 2).contiguous()
        K = self.A + beta[:, None, None] * torch.bmm(JT, self.J)
        pad = torch.ones(self.n_sub * self.nm, dtype=torch.float64, device="cuda")
        pad[self.dof] = 0.0
        K.diagonal(dim1=1, dim2=2).add_(pad.view(self.n_sub, self.nm))
        G = torch.linalg.solve(K, torch.cat([JT, self.b[:, :, None]], 2))
        c = G[:, :, -1].contiguous()
        G = G[:, :, :-1].contiguous()
        H = torch.bmm(self.J, G)
        d = torch.bmm(self.J, c[:, :, None])[:, :, 0]
        wp = torch.zeros(self.n_sub * self.cm, dtype=torch.float64, device="cuda")

        def fill(w):
            wp[self.slot] = w
            return wp.view(self.n_sub, self.cm, 1)

        return _admm(self.sl, beta, lambda w: (d + torch.bmm(H, fill(w))[:, :, 0]).reshape(-1)[self.slot],
                     lambda w: (c + torch.bmm(G, fill(w))[:, :, 0]).reshape(-1)[self.dof], e, iters, tol, z0, u0)


def _cross(a, b):
    return torch.linalg.cross(a, b, dim=-1)


def _mv(M, v):
    return (M * v[..., None, :]).sum(-1)


def _rot_log(Q):
    ang = torch.arccos(((Q.diagonal(dim1=-2, dim2=-1).sum(-1) - 1.0) / 2.0).clamp(-1.0, 1.0))
    f = torch.where(ang < 1e-4, 1.0 + ang * ang / 6.0, ang / torch.sin(ang).clamp(min=1e-300))
    v = torch.stack([Q[..., 2, 1] - Q[..., 1, 2], Q[..., 0, 2] - Q[..., 2, 0], Q[..., 1, 0] - Q[..., 0, 1]], -1)
    return 0.5 * f[..., None] * v


def _rot_exp(phi):
    return torch.linalg.matrix_exp(torch.stack([
        torch.stack([torch.zeros_like(phi[:, 0]), -phi[:, 2], phi[:, 1]], -1),
        torch.stack([phi[:, 2], torch.zeros_like(phi[:, 0]), -phi[:, 0]], -1),
        torch.stack([-phi[:, 1], phi[:, 0], torch.zeros_like(phi[:, 0])], -1)], -2))


class _Rigid:
    """Maximal-coordinate rigid bodies: construction, solve and state update of one step."""

    def __init__(self, sc):
        self.sc, self.sl = sc, _Slots(sc)
        self.mass, self.inertia = _f64(sc.mass), _f64(sc.inertia)
        self.sub, self.local = _i64(sc.body_sub), _i64(sc.body_local)

    def _rows(self, pd, j, m, k, body, lin, ang, sign):
        """Adds sign (lin, ang) of `body` to row k of interface j, member m."""
        g = self.sl.start[j, np.where(self.sc.if_nsub[j] > 1, m, 0)] + k
        J = pd.J.view(pd.n_sub, pd.cm, pd.nm // 6, 6)
        at = (_i64(self.sl.sub_np[g]), _i64(self.sl.loc_np[g]), _i64(self.sc.body_local[body]))
        J.index_put_(at, sign * torch.cat([lin, ang], -1), accumulate=True)

    def step(self, pos, R, vel, om, rho, iters, tol, z0, u0):
        sc, sl = self.sc, self.sl
        t = float(sc.dt)
        pd = _Padded(sc, sl)
        A = pd.A.view(pd.n_sub, pd.nm // 6, 6, pd.nm // 6, 6)
        Md = torch.cat([self.mass[:, None].expand(-1, 3), self.inertia], 1) * (2.0 / t)
        for c in range(6):
            A[self.sub, self.local, c, self.local, c] = Md[:, c]
        bb = torch.cat([Md[:, :3] * vel, Md[:, 3:] * om - _cross(om, self.inertia * om)], 1)
        bb[:, 2] -= self.mass * sc.gravity
        b = pd.b.view(pd.n_sub, pd.nm // 6, 6)
        b[self.sub, self.local] = bb
        e = torch.zeros(int(sl.row0[-1]), dtype=torch.float64, device="cuda")
        RT = R.transpose(1, 2)
        eye = torch.eye(3, dtype=torch.float64, device="cuda")
        gam = sc.baumgarte / t
        if len(sc.joint_body):
            a, bd, j = sc.joint_body[:, 0], sc.joint_body[:, 1], sc.joint_if
            ia, ib = _i64(a), _i64(bd)
            ra, rb, F, hb = _f64(sc.joint_anchor[:, 0]), _f64(sc.joint_anchor[:, 1]), _f64(sc.joint_frame_a), _f64(sc.joint_axis_b)
            sep = pos[ia] + _mv(R[ia], ra) - pos[ib] - _mv(R[ib], rb)
            cr = _cross(_mv(R[ib], hb), _mv(R[ia], F[:, 0]))
            zero = torch.zeros_like(ra)
            for k in range(5):
                d = eye[k].expand_as(ra) if k < 3 else _mv(R[ia], F[:, k - 2])
                for m, (bo, i, r, sg) in enumerate(((a, ia, ra, 1.0), (bd, ib, rb, -1.0))):
                    loc = _mv(RT[i], d)
                    self._rows(pd, j, m, k, bo, d if k < 3 else zero, _cross(r, loc) if k < 3 else loc, sg)
                e[_i64(sl.row0[j] + k)] = gam * (sep[:, k] if k < 3 else (d * cr).sum(-1))
        if len(sc.contact_body):
            c, j = sc.contact_body, sc.contact_if
            ic, r = _i64(c), _f64(sc.contact_point)
            for k, ax in enumerate((2, 0, 1)):
                d = eye[ax].expand_as(r)
                self._rows(pd, j, np.zeros_like(j), k, c, d, _cross(r, _mv(RT[ic], d)), 1.0)
            e[_i64(sl.row0[j])] = (pos[ic, 2] + _mv(R[ic], r)[:, 2]) / t
        self._links(pd, A, b, e, pos, R, t, gam)
        vh, lam, z, u = pd.solve(e, rho, iters, tol, z0, u0)
        bv = torch.zeros(pd.n_sub * pd.nm, dtype=torch.float64, device="cuda")
        bv[pd.dof] = vh
        bv = bv.view(pd.n_sub, pd.nm // 6, 6)[self.sub, self.local]
        return (pos + t * bv[:, :3], torch.bmm(R, _rot_exp(t * bv[:, 3:])), 2.0 * bv[:, :3] - vel,
                2.0 * bv[:, 3:] - om), vh, lam, z, u

    def _links(self, pd, A, b, e, pos, R, t, gam):
        sc, sl = self.sc, self.sl
        RT = R.transpose(1, 2)
        eye = torch.eye(3, dtype=torch.float64, device="cuda")
        for ty in (0, 1, 2):
            for two in (False, True):
                q = np.nonzero((sc.link_type == ty) & ((sc.link_body[:, 1] >= 0) == two))[0]
                if not len(q):
                    continue
                a, bd, j = sc.link_body[q, 0], sc.link_body[q, 1], sc.link_if[q]
                ia, ib = _i64(a), _i64(np.maximum(bd, 0))
                ra, rb, F = _f64(sc.link_anchor[q, 0]), _f64(sc.link_anchor[q, 1]), _f64(sc.link_frame[q])
                if ty == 2 and two:
                    n = pos[ia] - pos[ib]
                    ln = n.norm(dim=1)
                    n = n / ln[:, None]
                    phi0 = ln - ra[:, 0] - rb[:, 0]
                    t1 = eye[n.abs().argmin(1)]
                    t1 = t1 - (t1 * n).sum(-1, keepdim=True) * n
                    t1 = t1 / t1.norm(dim=1, keepdim=True)
                    dirs = [n, t1, _cross(n, t1)]
                elif ty == 2:
                    dirs = [F[:, 0], F[:, 1], F[:, 2]]
                    phi0 = (dirs[0] * pos[ia]).sum(-1) - rb[:, 0] - ra[:, 0]
                else:
                    dirs = [_mv(R[ia], F[:, k]) for k in range(3)]
                    if ty == 0:
                        sep = pos[ia] + _mv(R[ia], ra) - pos[ib] - _mv(R[ib], rb)
                    else:
                        log = _rot_log(torch.bmm(RT[ia], R[ib]))
                for k in range(3):
                    use = np.nonzero(sc.link_dim[q] > k)[0]
                    if not len(use):
                        continue
                    iu = _i64(use)
                    d = dirs[k][iu]
                    if ty == 2:
                        phi = phi0[iu]
                        pa, pb = -ra[iu, :1] * dirs[0][iu], rb[iu, :1] * dirs[0][iu]
                        rows = [(d, _mv(RT[ia[iu]], _cross(pa, d))), (d, _mv(RT[ib[iu]], _cross(pb, d)))]
                    elif ty == 0:
                        phi = (sep[iu] * d).sum(-1)
                        rows = [(d, _cross(ra[iu], F[iu, k])), (d, _cross(rb[iu], _mv(RT[ib[iu]], d)))]
                    else:
                        phi = -(F[iu, k] * log[iu]).sum(-1)
                        rows = [(torch.zeros_like(d), F[iu, k]), (torch.zeros_like(d), _mv(RT[ib[iu]], d))]
                    if not two and ty < 2:
                        phi = torch.zeros_like(phi)
                    own = j[use] >= 0
                    h = np.nonzero(own)[0]
                    if len(h):
                        jh, ih = j[use][h], _i64(h)
                        self._rows(pd, jh, np.zeros_like(jh), k, a[use][h], rows[0][0][ih], rows[0][1][ih], 1.0)
                        if two:
                            self._rows(pd, jh, np.ones_like(jh), k, bd[use][h], rows[1][0][ih], rows[1][1][ih], -1.0)
                        kd = _i64(sc.if_kind[jh])
                        ek = torch.where(kd == 3, phi[ih], torch.where(kd == 1, phi[ih] / t if k == 0 else 0.0 * phi[ih],
                                                                       gam * phi[ih]))
                        e[_i64(sl.row0[jh] + k)] = ek
                    f = np.nonzero(~own)[0]
                    if len(f):
                        # folded soft rows: A += k alpha J^T J, b -= k J^T phi
                        i_f, qf = _i64(f), q[use][f]
                        kk, al = _f64(sc.link_k[qf])[:, None], _f64(sc.link_alpha[qf])[:, None]
                        sub = self.sub[ia[iu][i_f]]
                        la, lb = self.local[ia[iu][i_f]], self.local[ib[iu][i_f]]
                        Ja, Jb = torch.cat([r[i_f] for r in rows[0]], -1), -torch.cat([r[i_f] for r in rows[1]], -1)
                        for l1, J1 in ((la, Ja), (lb, Jb)):
                            b.index_put_((sub, l1), -kk * phi[i_f][:, None] * J1, accumulate=True)
                            for l2, J2 in ((la, Ja), (lb, Jb)):
                                # A viewed as (subsystem, block, 6, block, 6)
                                blk = (kk * al)[:, :, None] * J1[:, :, None] * J2[:, None, :]
                                A.permute(0, 1, 3, 2, 4).index_put_((sub, l1, l2), blk, accumulate=True)


def _fem_step(fs, pos, vel, iters, tol):
    sl = _Slots(fs)
    t, lib = float(fs.dt), torch.linalg
    ns, nn = fs.n_sub, fs.n_nodes
    tets, rest = _i64(fs.tets), _f64(fs.rest)
    tsub = _i64(fs.tet_sub)
    X, x = rest[tets], pos[tets]
    D = (X[:, 1:] - X[:, :1]).transpose(1, 2)          # columns X_a - X_0
    V = lib.det(D) / 6.0
    g = lib.inv(D)                                      # rows g_1..g_3
    g = torch.cat([-g.sum(1, keepdim=True), g], 1)      # (nt, 4, 3)
    nu, E = _f64(fs.poisson), _f64(fs.young)
    lam, mu = (E * nu / ((1 + nu) * (1 - 2 * nu)))[tsub], (E / (2 * (1 + nu)))[tsub]
    mass = torch.zeros(nn, dtype=torch.float64, device="cuda").index_add_(
        0, tets.reshape(-1), (fs.density * V / 4.0)[:, None].expand(-1, 4).reshape(-1))
    R = torch.bmm(x.transpose(1, 2), g)
    for _ in range(12):
        R = 0.5 * (R + lib.inv(R).transpose(1, 2))
    G = torch.bmm((torch.bmm(x, R) - X).transpose(1, 2), g)
    eye = torch.eye(3, dtype=torch.float64, device="cuda")
    P = V[:, None, None] * (lam[:, None, None] * G.diagonal(dim1=1, dim2=2).sum(1)[:, None, None] * eye +
                            mu[:, None, None] * (G + G.transpose(1, 2)))
    f = -torch.bmm(torch.bmm(R, P), g.transpose(1, 2)).transpose(1, 2)   # (nt, 4, 3)
    b = (2.0 / t) * mass[:, None] * vel
    b.index_add_(0, tets.reshape(-1), f.reshape(-1, 3))
    b[:, 2] -= mass * fs.gravity
    m = int(fs.sub_nodes.max())
    off = _i64(fs.node_off)
    loc = tets - off[tsub][:, None]
    A = torch.zeros(ns, m, m, 3, 3, dtype=torch.float64, device="cuda")
    rg = torch.bmm(g, R.transpose(1, 2))                # rows R g_a
    for a in range(4):
        for c in range(4):
            K = (lam[:, None, None] * rg[:, a, :, None] * rg[:, c, None, :] +
                 mu[:, None, None] * rg[:, c, :, None] * rg[:, a, None, :] +
                 (mu * (g[:, a] * g[:, c]).sum(-1))[:, None, None] * eye) * V[:, None, None]
            A.index_put_((tsub, loc[:, a], loc[:, c]), 0.5 * t * K, accumulate=True)
    nsub = _i64(np.repeat(np.arange(ns), fs.sub_nodes))
    nloc = torch.arange(nn, device="cuda") - off[nsub]
    for c in range(3):
        A[nsub, nloc, nloc, c, c] += (2.0 / t) * mass
    n = 3 * m
    A = A.permute(0, 1, 3, 2, 4).reshape(ns, n, n)
    # every slot row selects one DOF: a tie +-1 on the node's axis, a contact (z, x, y)
    mem, row = np.zeros(sl.n, np.int64), np.zeros(sl.n, np.int64)
    jj = np.zeros(sl.n, np.int64)
    for j in range(fs.n_if):
        for q in range(int(fs.if_nsub[j])):
            s = sl.start[j, q]
            jj[s:s + 3], mem[s:s + 3], row[s:s + 3] = j, q, (0, 1, 2)
    con = fs.if_kind[jj] == 1
    axis = np.where(con, (row + 2) % 3, row)
    node = fs.if_node[jj, mem]
    col = _i64(sl.sub_np * n + 3 * (node - fs.node_off[sl.sub_np]) + axis)
    sign = _f64(np.where(mem == 1, -1.0, 1.0))
    beta = A.diagonal(dim1=1, dim2=2).sum(1) / _f64(np.maximum(sl.nc, 1))
    beta = torch.where(_i64(sl.nc) > 0, beta, torch.ones_like(beta))
    cnt = torch.zeros(ns * n, dtype=torch.float64, device="cuda").index_add_(0, col, torch.ones_like(sign))
    K = A + torch.diag_embed(beta[:, None] * cnt.view(ns, n))
    bp = torch.zeros(ns, m, 3, dtype=torch.float64, device="cuda")
    bp[nsub, nloc] = b
    bp = bp.view(ns, n, 1)
    Ki = torch.cat([lib.inv(k) for k in K.split(32)])

    def v_all(w):
        r = torch.zeros(ns * n, dtype=torch.float64, device="cuda").index_add_(0, col, sign * w)
        return torch.bmm(Ki, bp + r.view(ns, n, 1)).reshape(-1)

    dof = ((nsub * n + 3 * nloc)[:, None] + torch.arange(3, device="cuda")).reshape(-1)
    j0, two = np.arange(fs.n_if), fs.if_nsub > 1
    e = torch.zeros(fs.n_if, 3, dtype=torch.float64, device="cuda")
    if two.any():
        e[_i64(j0[two])] = fs.baumgarte / t * (pos[_i64(fs.if_node[two, 0])] - pos[_i64(fs.if_node[two, 1])])
    if (~two).any():
        e[_i64(j0[~two]), 0] = pos[_i64(fs.if_node[~two, 0]), 2] / t
    vh, lam_, _, _ = _admm(sl, beta, lambda w: sign * v_all(w)[col], lambda w: v_all(w)[dof], e.reshape(-1), iters, tol)
    v3 = vh.view(-1, 3)
    return pos + t * v3, 2.0 * v3 - vel, vh, lam_


def _mlp_exact(case, seed):
    w, params, x, target, wt, scale, shift = (v if isinstance(v, list) else v.double() for v in _mlp_inputs(case, seed))
    W, B, at = [], [], 0
    for a, c in zip(w[:-1], w[1:]):
        W.append(params[at:at + a * c].view(c, a))
        B.append(params[at + a * c:at + a * c + c])
        at += a * c + c
    h = [x * scale + shift]
    for k in range(len(W)):
        y = h[-1] @ W[k].t() + B[k]
        h.append(y.clamp(min=0.0) if k + 1 < len(W) else y)
    if not case["train"]:
        return h[-1]
    r = h[-1] - target
    d = wt * r
    grads = []
    for k in reversed(range(len(W))):
        grads = [(d.t() @ h[k]).reshape(-1), d.sum(0)] + grads
        d = (d @ W[k]) * (h[k] > 0)
    return {"y": h[-1], "loss": (0.5 * wt * r * r).sum().reshape(1), "grad": torch.cat(grads)}


def exact(case, seed):
    if case["kind"] == "mlp":
        return _mlp_exact(case, seed)
    dt = DTYPES[case["dtype"]]
    given = lambda a: _f64(a).to(dt).double()  # the values the library is handed  # noqa: E731
    if case["kind"] == "solve":
        p, A, b, J, e = _solve_inputs(case, seed)
        sl = _Slots(p)
        pd = _Padded(p, sl)
        A, J = given(A), given(J)
        n, nc = pd.n, sl.nc
        a0, j0 = np.concatenate([[0], np.cumsum(n * n)]), np.concatenate([[0], np.cumsum(nc * n)])
        for i in range(p.n_sub):
            pd.A[i, :n[i], :n[i]] = A[a0[i]:a0[i + 1]].view(n[i], n[i])
            pd.J[i, :nc[i], :n[i]] = J[j0[i]:j0[i + 1]].view(nc[i], n[i])
        pd.b.view(-1)[pd.dof] = given(b)
        vh, lam, z, u = pd.solve(given(e), 0.0, case["iters"], case["tol"])
        return {"v_hat": vh, "lam": lam, "z": z, "u": u}
    if case["kind"] == "fem":
        fs, pos, vel = _fem_state(case, seed)
        pos, vel, vh, lam = _fem_step(fs, given(pos), given(vel), case["iters"], case["tol"])
        return {"state": [pos.reshape(-1), vel.reshape(-1)], "v_hat": vh, "lam": lam}
    sc, *state = _rigid_state(case, seed)
    rg = _Rigid(sc)
    state, z, u = [given(a) for a in state], None, None
    for _ in range(case["steps"]):
        state, vh, lam, z, u = rg.step(*state, case["rho"], case["iters"], case["tol"], z, u)
    return {"state": [a.reshape(-1) for a in state], "v_hat": vh, "lam": lam}
