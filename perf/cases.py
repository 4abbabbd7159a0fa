"""Performance cases: the library's batched solvers as a user's program calls them.

Every case is a dict of plain values.  ``prepare`` builds what the program has in
hand before the call (context, uploaded robot, inputs and output buffers on the
GPU, a trained seeder), ``run`` makes one pass through the package's entry points
and returns every output, ``work`` gives the bytes and FLOPs a pass cannot do
without and ``exact`` the outputs in 64 bits where they are well defined.

Robots and draws follow the repository's synthetic workloads: serial arms with
axes z, y, z, ... and link offsets (U[0.05, 0.30], 0, U[0.05, 0.30]), limits
+-U[pi/2, pi]; a planar base under the 7-joint arm; a four-fingered hand; a
34-joint tree.  Targets are the poses of uniform in-limit configurations, so
they are reachable; seeds are uniform in-limit configurations.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2505_03728_amd as pk
from paper_2505_03728_amd.flops import lm_flops

DEV = "cuda:0"
AX = {"x": (1.0, 0.0, 0.0), "y": (0.0, 1.0, 0.0), "z": (0.0, 0.0, 1.0)}


# ----------------------------------------------------------------- robots

def f32(a):
    """FP32-rounded, as float64."""
    return np.asarray(a, np.float32).astype(np.float64)


def tree(parent, axes, offset, lim, ee_joint, ee_offset, kind, mount=None, types=None):
    n, m = len(parent), len(ee_joint)
    ident = [1.0, 0.0, 0.0, 0.0]
    return SimpleNamespace(
        parent=np.asarray(parent, np.int32), axis=f32([AX[a] for a in axes]),
        offset=f32(offset), mount_quat=f32(mount if mount is not None else [ident] * n),
        lower=-f32(lim), upper=f32(lim), ee_joint=np.asarray(ee_joint, np.int32),
        ee_offset=f32(ee_offset), ee_quat=f32([ident] * m), ee_kind=np.full(m, kind, np.int32),
        joint_type=None if types is None else np.asarray(types, np.int32))


def offsets(rng, count, lo, hi):
    out = np.zeros((count, 3))
    out[:, [0, 2]] = rng.uniform(lo, hi, (count, 2))
    return out


def arm(n, kind=pk.EE_POSE):
    rng = np.random.default_rng(100 + n)
    off, lim = offsets(rng, n + 1, 0.05, 0.30), rng.uniform(math.pi / 2, math.pi, n)
    return tree(range(-1, n - 1), ("zy" * n)[:n], off[:n], lim, [n - 1], off[n:], kind)


def mobile10():
    """SE(2) base (x, y, yaw) carrying the 7-joint arm."""
    a = arm(7)
    return tree(range(-1, 9), "xyz" + "zyzyzyz", np.vstack([np.zeros((3, 3)), a.offset]),
                [2.0, 2.0, math.pi, *a.upper], [9], a.ee_offset, pk.EE_POSE,
                types=[1, 1, 0] + [0] * 7)


def hand16():
    """Four fingers of four joints, a position target per fingertip."""
    rng = np.random.default_rng(16)
    off, tip = offsets(rng, 16, 0.02, 0.05), offsets(rng, 4, 0.02, 0.05)
    off[0::4, 1] += (np.arange(4) - 1.5) * 0.02
    parent = [-1 if j % 4 == 0 else j - 1 for j in range(16)]
    return tree(parent, "zyzy" * 4, off, rng.uniform(math.pi / 2, math.pi, 16), [3, 7, 11, 15], tip,
                pk.EE_POSITION)


def tree34():
    """Six-joint torso and four seven-joint branches, a pose target per branch."""
    rng = np.random.default_rng(34)
    off, tip = offsets(rng, 34, 0.05, 0.30), offsets(rng, 4, 0.05, 0.30)
    parent = list(range(-1, 5)) + [5 if i == 0 else 6 + 7 * c + i - 1 for c in range(4) for i in range(7)]
    mount = np.tile([1.0, 0.0, 0.0, 0.0], (34, 1))
    for c in range(4):
        mount[6 + 7 * c] = [math.cos(c * math.pi / 4), 0.0, 0.0, math.sin(c * math.pi / 4)]
    return tree(parent, "zyzyzy" + "zyzyzyz" * 4, off, rng.uniform(math.pi / 2, math.pi, 34),
                [12, 19, 26, 33], tip, pk.EE_POSE, mount=mount)


def robot(name):
    if name.startswith("arm"):
        return arm(int(name[3:].rstrip("p")), pk.EE_POSITION if name.endswith("p") else pk.EE_POSE)
    return {"mobile10": mobile10, "hand16": hand16, "tree34": tree34}[name]()


# ------------------------------------------------- FP64 kinematics (torch)

def rot_of_quat(q):
    q = q / q.norm(dim=-1, keepdim=True)
    w, x, y, z = q.unbind(-1)
    return torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                        2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                        2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)],
                       -1).unflatten(-1, (3, 3))


def quat_of_rot(R):
    """Unit quaternion with w >= 0: the column of the largest component of 4 q q^T."""
    t = R[..., 0, 0], R[..., 1, 1], R[..., 2, 2]
    a, b, c = R[..., 2, 1] - R[..., 1, 2], R[..., 0, 2] - R[..., 2, 0], R[..., 1, 0] - R[..., 0, 1]
    d, e, f = R[..., 0, 1] + R[..., 1, 0], R[..., 0, 2] + R[..., 2, 0], R[..., 1, 2] + R[..., 2, 1]
    M = torch.stack([1 + t[0] + t[1] + t[2], a, b, c, a, 1 + t[0] - t[1] - t[2], d, e,
                     b, d, 1 - t[0] + t[1] - t[2], f, c, e, f, 1 - t[0] - t[1] + t[2]],
                    -1).unflatten(-1, (4, 4))
    k = M.diagonal(dim1=-2, dim2=-1).argmax(-1)
    q = torch.gather(M, -2, k[..., None, None].expand(*k.shape, 1, 4)).squeeze(-2)
    q = q / q.norm(dim=-1, keepdim=True)
    return torch.where(q[..., :1] < 0, -q, q)


def mm(A, B):
    """Batched 3 x 3 products, elementwise (any batch size)."""
    return (A.unsqueeze(-1) * B.unsqueeze(-3)).sum(-2)


def mv(A, x):
    return (A * x.unsqueeze(-2)).sum(-1)


def fk64(tr, q):
    """q [N, n] float64 -> per EE (p [N, 3], R [N, 3, 3])."""
    t = lambda a: torch.as_tensor(np.asarray(a, np.float64), device=q.device)
    mount, ax, off = rot_of_quat(t(tr.mount_quat)), t(tr.axis), t(tr.offset)
    ee_q, ee_o = rot_of_quat(t(tr.ee_quat)), t(tr.ee_offset)
    frames = []
    eye = torch.eye(3, dtype=q.dtype, device=q.device)
    for j, par in enumerate(tr.parent):
        p, R = frames[par] if par >= 0 else (torch.zeros_like(q[:, :3]), eye.expand(len(q), 3, 3))
        p, R = p + mv(R, off[j].expand(len(q), 3)), mm(R, mount[j].expand(len(q), 3, 3))
        x = q[:, j, None]
        if tr.joint_type is not None and tr.joint_type[j] == 1:
            p = p + mv(R, ax[j] * x)
        else:
            h = 0.5 * x
            R = mm(R, rot_of_quat(torch.cat([h.cos(), h.sin() * ax[j]], -1)))
        frames.append((p, R))
    out = []
    for k, e in enumerate(tr.ee_joint):
        p, R = frames[e]
        out.append((p + mv(R, ee_o[k].expand(len(q), 3)), mm(R, ee_q[k].expand(len(q), 3, 3))))
    return out


def poses64(tr, q):
    """[m][N, 7]: positions and quaternions."""
    return [torch.cat([p, quat_of_rot(R)], -1) for p, R in fk64(tr, q)]


# ------------------------------------------------------------------ inputs

def generator(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * int(seed) + stream)
    return g


def configs(tr, count, g):
    """[n, count] uniform in-limit configurations (FP32)."""
    lo = torch.as_tensor(tr.lower, dtype=torch.float32, device=DEV)[:, None]
    hi = torch.as_tensor(tr.upper, dtype=torch.float32, device=DEV)[:, None]
    return lo + (hi - lo) * torch.rand((len(tr.lower), count), generator=g, device=DEV)


def target_planes(tr, q):
    """Target planes [floats, T] of configurations q [n, T]."""
    planes = [p[:, :7 if k == pk.EE_POSE else 3].T for p, k in zip(poses64(tr, q.double().T), tr.ee_kind)]
    return torch.cat(planes).float().contiguous()


def lm_options(c, iters=None):
    mob = c.get("robot") == "mobile10"
    return pk.Options(max_iters=c["iters"] if iters is None else iters, early_exit=c["early_exit"],
                      tol_pos=5e-3 if mob else 1e-3, tol_rot=5e-2 if mob else 1e-2)


def ik_inputs(c, tr, seed, T, K):
    q = configs(tr, T, generator(seed, 1))
    s = configs(tr, T * K, generator(seed, 2))
    if c.get("robot") == "mobile10":     # the base starts at the origin, targets within 1 m of it
        q[:3] *= torch.tensor([0.5, 0.5, 0.0], device=DEV)[:, None]
        s[:3] = 0.0
    return target_planes(tr, q), s.contiguous()


# ---------------------------------------------------------------- the cases

def listed():
    return [
        # one target, eight seeds: a control loop's call, all latency
        {"name": "ik_arm7_1x8", "kind": "ik", "robot": "arm7", "T": 1, "K": 8, "iters": 30, "early_exit": True,
         "w_rest": 0.01, "best": True},
        # the benchmark batch
        {"name": "ik_arm7_16384x8", "kind": "ik", "robot": "arm7", "T": 16384, "K": 8, "iters": 30,
         "early_exit": True, "w_rest": 0.01, "best": True},
        # an odd batch: six joints, five seeds (a target's seeds straddle wavefronts), no early exit
        {"name": "ik_arm6_1237x5", "kind": "ik", "robot": "arm6", "T": 1237, "K": 5, "iters": 30,
         "early_exit": False, "w_rest": 0.0, "best": True},
        # whole-body IK of a 34-joint tree with four pose targets
        {"name": "ik_tree34_4096x1", "kind": "ik", "robot": "tree34", "T": 4096, "K": 1, "iters": 40,
         "early_exit": False, "w_rest": 0.0, "best": False},
        # mobile base (two sliding joints) under the arm
        {"name": "ik_mobile10_4096x4", "kind": "ik", "robot": "mobile10", "T": 4096, "K": 4, "iters": 30,
         "early_exit": True, "w_rest": 0.01, "best": True},
        # several robots in one scheduled call
        {"name": "mixed_84k", "kind": "mixed", "arm": 60000, "hand": 20000, "tree": 4096, "iters": 50,
         "early_exit": True},
        # beam search over 64 seeds per target
        {"name": "beam_1000x64", "kind": "beam", "T": 1000, "seeds": 64, "iters0": 6, "keep": 4, "iters1": 10,
         "early_exit": False},
        # the whole learned-seed pipeline: network, refinement, restart, random fallback
        {"name": "seeded_131072", "kind": "seeded", "T": 131072, "hidden": 512, "fallback": 128},
        # a stretch of seeder training (64 steps)
        {"name": "train_64x8192", "kind": "train", "steps": 64, "batch": 8192, "hidden": 512, "depth": 3, "K": 8},
        # a planner's batch of trajectories
        {"name": "traj_1024x32x7", "kind": "traj", "B": 1024, "T": 32, "n": 7, "iters": 20, "early_exit": False},
        # a few trajectories of odd length
        {"name": "traj_37x25x6", "kind": "traj", "B": 37, "T": 25, "n": 6, "iters": 20, "early_exit": False},
        # forward kinematics of a large sample (building training targets, checking solutions)
        {"name": "fk_arm7_1000003", "kind": "fk", "robot": "arm7", "N": 1000003, "frames": False},
    ]


def log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["ik"] * 4 + ["mixed", "beam", "seeded", "train", "traj", "traj", "fk"])
    if kind == "ik":
        name = rng.choice(["arm7", "arm7", "mobile10", "hand16", "tree34", "arm%d" % rng.randint(2, 10),
                           "arm%dp" % rng.randint(3, 8)])
        K = rng.choice([1, 1, 2, 3, 4, 5, 8, 8, 16]) if name != "tree34" else rng.choice([1, 2])
        N = log_int(rng, 8, {"tree34": 4096, "hand16": 20000, "mobile10": 32768}.get(name, 131072))
        return {"kind": kind, "robot": name, "T": max(1, N // K), "K": K, "iters": rng.randint(10, 50),
                "early_exit": rng.random() < 0.6, "w_rest": rng.choice([0.0, 0.01]), "best": rng.random() < 0.7}
    if kind == "mixed":
        return {"kind": kind, "arm": log_int(rng, 100, 60000), "hand": log_int(rng, 100, 20000),
                "tree": log_int(rng, 20, 4096), "iters": rng.randint(20, 50), "early_exit": True}
    if kind == "beam":
        return {"kind": kind, "T": log_int(rng, 1, 2000), "seeds": rng.choice([64, 64, 48, 32]), "iters0": 6,
                "keep": rng.choice([3, 4, 4, 8]), "iters1": 10, "early_exit": rng.random() < 0.5}
    if kind == "seeded":
        return {"kind": kind, "T": log_int(rng, 500, 131072), "hidden": rng.choice([256, 512]),
                "fallback": rng.choice([32, 64, 128])}
    if kind == "train":
        return {"kind": kind, "steps": rng.randint(8, 64), "batch": 128 * log_int(rng, 8, 64),
                "hidden": rng.choice([256, 512]), "depth": rng.choice([2, 3]), "K": rng.choice([4, 8])}
    if kind == "traj":
        n = rng.choice([4, 6, 7, 7, 10])
        return {"kind": kind, "B": log_int(rng, 1, 1024), "T": rng.randint(8, min(36, 256 // n)), "n": n,
                "iters": rng.randint(10, 20), "early_exit": rng.random() < 0.3}
    return {"kind": kind, "robot": rng.choice(["arm7", "arm%d" % rng.randint(2, 10), "mobile10", "hand16", "tree34"]),
            "N": log_int(rng, 1000, 300000), "frames": rng.random() < 0.3}


# ------------------------------------------------------------------ prepare

TRAJ_COSTS = {"dt": 0.05, "w_pos": 10.0, "w_rot": 5.0, "w_limit": 10.0, "w_smooth": 0.1, "w_vel": 1.0,
              "w_acc": 0.05, "w_jerk": 0.01}
VMAX = 2.0
LR = 1e-3


def net_init(sizes, seed):
    """[(W, b)] per layer, U(+-1/sqrt(fan in))."""
    rng = np.random.default_rng([int(seed), 3])
    return [(rng.uniform(-1, 1, (o, i)).astype(np.float32) / np.float32(math.sqrt(i)),
             rng.uniform(-1, 1, o).astype(np.float32) / np.float32(math.sqrt(i)))
            for i, o in zip(sizes[:-1], sizes[1:])]


def train_inputs(c, seed):
    tr = arm(7)
    S = c["steps"] * c["batch"]
    q = configs(tr, S, generator(seed, 5)).contiguous()
    perm = torch.randperm(S, generator=generator(seed, 6), device=DEV).to(torch.int32)[None].contiguous()
    return tr, q, perm, net_init([7] + [c["hidden"]] * c["depth"] + [7 * c["K"]], seed)


def traj_inputs(c, seed):
    """As a planner would start: straight line between perturbed end configurations plus a bump."""
    tr, B, T, n = arm(c["n"]), c["B"], c["T"], c["n"]
    g = generator(seed, 7)
    qa, qb = configs(tr, B, g), configs(tr, B, g)
    ea, eb, u = torch.randn((3, B, n), generator=g, device=DEV)
    s = torch.linspace(0, 1, T, device=DEV)[None, :, None]
    init = ((1 - s) * (qa.T + 0.05 * ea)[:, None] + s * (qb.T + 0.05 * eb)[:, None] +
            0.3 * torch.sin(math.pi * s) * (u / u.norm(dim=1, keepdim=True))[:, None])
    return tr, target_planes(tr, qa), target_planes(tr, qb), init.contiguous()


def prepare(case, seed):
    c, st = case, SimpleNamespace(case=case)
    kind = c["kind"]
    ctx = st.ctx = pk.Context(0)
    if kind == "ik":
        tr = robot(c["robot"])
        st.rid = ctx.upload(tr)
        st.targets, st.seeds = ik_inputs(c, tr, seed, c["T"], c["K"])
        st.w = pk.Weights(w_pos=10.0 if c["robot"] == "hand16" else 1.0, w_rest=c["w_rest"])
        st.o = lm_options(c)
        st.out = ctx.alloc_outputs(st.rid, c["T"], c["K"], best=c["best"])
    elif kind == "mixed":
        st.groups = []
        for i, (name, T) in enumerate([("arm7", c["arm"]), ("hand16", c["hand"]), ("tree34", c["tree"])]):
            tr = robot(name)
            rid = ctx.upload(tr)
            tg, s = ik_inputs(c, tr, 3 * seed + i, T, 1)
            out = ctx.alloc_outputs(rid, T, 1)
            del out["pose_cost"]         # the scheduler does not report it
            st.groups.append({"rid": rid, "targets": tg, "seeds": s, "K": 1, "out": out,
                              "weights": pk.Weights(w_pos=10.0 if name == "hand16" else 1.0, w_rest=0.01)})
        st.o = lm_options(c)
    elif kind == "beam":
        tr = arm(7)
        st.rid = ctx.upload(tr)
        st.targets, st.seeds = ik_inputs(c, tr, seed, c["T"], c["seeds"])
        st.w, st.o = pk.Weights(), lm_options(c, 16)
        st.out = ctx.alloc_beam_outputs(st.rid, c["T"], c["seeds"], c["keep"])
    elif kind == "seeded":
        # a seeder trained for 192 steps: most targets end in the refinement, a good share in the
        # restart, some in the fallback
        tr, q, perm, init = train_inputs({"steps": 192, "batch": 8192, "hidden": c["hidden"], "depth": 3, "K": 8}, 1)
        st.rid = ctx.upload(tr)
        st.seeder = pk.Seeder(ctx, st.rid, K=8, hidden=c["hidden"], depth=3, init=init)
        st.seeder.train(q, batch=8192, epochs=1, lr=LR, perm=perm)
        st.targets = target_planes(tr, configs(tr, c["T"], generator(seed, 1)))
        st.fb = configs(tr, c["T"] * c["fallback"], generator(seed, 2)).contiguous()
        st.w = pk.Weights(w_rest=0.01)
        st.refine, st.o = pk.Options(max_iters=6, early_exit=True), pk.Options(max_iters=30, early_exit=True)
    elif kind == "train":
        tr, st.q, st.perm, init = train_inputs(c, seed)
        st.rid = ctx.upload(tr)
        st.seeder = pk.Seeder(ctx, st.rid, K=c["K"], hidden=c["hidden"], depth=c["depth"], init=init)
        st.loss = torch.zeros(c["steps"], dtype=torch.float32, device=DEV)
    elif kind == "traj":
        tr, st.start, st.goal, st.init = traj_inputs(c, seed)
        st.rid = ctx.upload(tr)
        st.vmax = torch.full((c["n"],), VMAX, dtype=torch.float32, device=DEV)
        st.o = pk.Options(max_iters=c["iters"], early_exit=c["early_exit"])
        st.out = None
    else:
        tr = robot(c["robot"])
        st.rid = ctx.upload(tr)
        st.q = configs(tr, c["N"], generator(seed, 8)).contiguous()
    return st


# ---------------------------------------------------------------------- run

def outputs(d):
    return {k: v for k, v in d.items() if not k.startswith("_")}


def run(st):
    c, ctx = st.case, st.ctx
    kind = c["kind"]
    if kind == "ik":
        return outputs(ctx.ik_solve(st.rid, st.targets, st.seeds, c["K"], st.w, st.o, st.out))
    if kind == "mixed":
        # the default schedule: every group in one persistent launch, on the caller's stream
        ctx.ik_solve_mixed(st.groups, st.o, waves_per_cu=8, use_graph=False)
        return [outputs(g["out"]) for g in st.groups]
    if kind == "beam":
        return ctx.ik_beam(st.rid, st.targets, st.seeds, st.w, st.o, n_seeds=c["seeds"], iters0=c["iters0"],
                           keep=c["keep"], iters1=c["iters1"], out=st.out)
    if kind == "seeded":
        return ctx.ik_solve_seeded(st.rid, st.targets, st.seeder, st.w, st.refine, fallback=st.o,
                                   fallback_seeds=st.fb, fallback_K=c["fallback"], restart_iters=20)
    if kind == "train":
        st.seeder.train(st.q, batch=c["batch"], epochs=1, lr=LR, perm=st.perm, loss_log=st.loss)
        return {"loss": st.loss, "params": st.seeder.get(0)}
    if kind == "traj":
        st.out = ctx.traj_solve(st.rid, st.start, st.goal, st.init, TRAJ_COSTS, st.o, vmax=st.vmax, out=st.out)
        return st.out
    r = ctx.fk(st.rid, st.q, frames=c["frames"])
    return list(r) if c["frames"] else r


# --------------------------------------------------------------------- work

def ik_work(name, T, K, iters, early, best=False, scalars=6):
    """Each input once, each output once; LM FLOPs with three trials in four accepted and, with
    early exit, half of the iteration budget used."""
    tr = robot(name)
    n, m, N = len(tr.parent), len(tr.ee_joint), T * K
    tf = sum(7 if k == pk.EE_POSE else 3 for k in tr.ee_kind)
    blocks = None if name == "tree34" else [4] * 4 if name == "hand16" else [n]
    its = N * iters * (0.5 if early else 1.0)
    return (4 * (tf * T + 2 * n * N + (2 * m + scalars) * N + ((n + 2) * T if best else 0)),
            lm_flops(tr.parent, tr.ee_joint, tr.ee_kind, blocks, its, 0.75 * its, N))


def net_flops(hidden, depth, K, rows):
    return 2.0 * rows * (7 * hidden + (depth - 1) * hidden * hidden + hidden * 7 * K)


def work(case):
    c = case
    kind = c["kind"]
    if kind == "ik":
        b, f = ik_work(c["robot"], c["T"], c["K"], c["iters"], c["early_exit"], c["best"])
    elif kind == "mixed":
        parts = [ik_work(r, c[k], 1, c["iters"], True) for r, k in
                 (("arm7", "arm"), ("hand16", "hand"), ("tree34", "tree"))]
        b, f = sum(p[0] for p in parts), sum(p[1] for p in parts)
    elif kind == "beam":
        T = c["T"]
        b = 4 * T * (7 + 7 * c["seeds"] + 7 + 5)
        f = (ik_work("arm7", T, c["seeds"], c["iters0"], c["early_exit"])[1] +
             ik_work("arm7", T, c["keep"], c["iters1"], c["early_exit"])[1])
    elif kind == "seeded":
        # refinement of the learned seeds; a fifth of the targets restarted, 2% in the fallback
        T = c["T"]
        f = net_flops(c["hidden"], 3, 8, T) + ik_work("arm7", T, 8, 6, False)[1]
        f += ik_work("arm7", T // 5, 8, 20, True)[1] + ik_work("arm7", T // 50, c["fallback"], 30, True)[1]
        b = 4 * T * (7 + 7 + 3) + 4 * 7 * (T // 50) * c["fallback"]
    elif kind == "train":
        S = c["steps"] * c["batch"]
        params = 7 * c["hidden"] + (c["depth"] - 1) * c["hidden"] ** 2 + c["hidden"] * 7 * c["K"]
        f = 3 * net_flops(c["hidden"], c["depth"], c["K"], S)
        b = S * 4 * 8 + c["steps"] * params * (3 * 8 + 2)     # samples; FP32 weights and moments, BF16 copies
    elif kind == "traj":
        V, hb = c["T"] * c["n"], 4 * c["n"]
        its = c["B"] * c["iters"] * (0.5 if c["early_exit"] else 1.0)
        f = its * V * (hb * (hb + 1) + hb + 4 * hb + 3)
        b = 4 * c["B"] * (2 * V + 14 + 8)
    else:
        tr = robot(c["robot"])
        n, m = len(tr.parent), len(tr.ee_joint)
        f = c["N"] * (36.0 * n + 50.0 * m)
        b = 4 * c["N"] * (n + 7 * m + (12 * n if c["frames"] else 0))
    return {"bytes": float(b), "flops": float(f)}


# -------------------------------------------------------------------- exact

def exact(case, seed):
    """64-bit outputs of the cases whose outputs have such a value.  An IK solution has none: the
    iterates of an LM run from a random seed part from any other rounding's after a rejected or a
    nearly singular step, so only its bits can be compared (ik, mixed, beam, seeded: None)."""
    return {"fk": exact_fk, "train": exact_train, "traj": exact_traj}.get(case["kind"], lambda *_: None)(case, seed)


def exact_fk(c, seed):
    tr = robot(c["robot"])
    q = configs(tr, c["N"], generator(seed, 8)).double().T
    ee = torch.stack([p.T for p in poses64(tr, q)])
    if not c["frames"]:
        return ee
    tips = SimpleNamespace(**{**tr.__dict__, "ee_joint": np.arange(len(tr.parent)),
                              "ee_offset": np.zeros((len(tr.parent), 3)),
                              "ee_quat": np.tile([1.0, 0, 0, 0], (len(tr.parent), 1))})
    fr = torch.stack([torch.cat([R.flatten(1), p], -1).T for p, R in fk64(tips, q)])
    return [ee, fr]


def exact_train(c, seed):
    """The same steps in float64: encoded poses, SiLU layers, closest-seed loss, Adam."""
    tr, q, perm, init = train_inputs(c, seed)
    K, B = c["K"], c["batch"]
    reach = float(np.linalg.norm(tr.offset, axis=1).sum() + np.linalg.norm(tr.ee_offset, axis=1).max())
    qa = q.double().T
    x = poses64(tr, qa)[0]
    x = torch.cat([x[:, :3] / reach, x[:, 3:]], -1)
    P = [torch.as_tensor(a, dtype=torch.float64, device=DEV).requires_grad_() for wb in init for a in wb]
    M, V, losses = [torch.zeros_like(p) for p in P], [torch.zeros_like(p) for p in P], []
    for t in range(c["steps"]):
        idx = perm[0, t * B:(t + 1) * B].long()
        h = x[idx]
        for i in range(0, len(P), 2):
            h = h @ P[i].T + P[i + 1]
            if i + 2 < len(P):
                h = h * torch.sigmoid(h)
        loss = (h.unflatten(1, (K, 7)) - qa[idx][:, None]).square().sum(-1).min(1).values.mean()
        losses.append(loss.detach())
        grads = torch.autograd.grad(loss, P)
        c1, c2 = 1 - 0.9 ** (t + 1), 1 - 0.999 ** (t + 1)
        with torch.no_grad():
            for p, g, m, v in zip(P, grads, M, V):
                m.mul_(0.9).add_(0.1 * g)
                v.mul_(0.999).add_(0.001 * g * g)
                p -= LR * (m / c1) / ((v / c2).sqrt() + 1e-8)
    return {"loss": torch.stack(losses), "params": [(P[i].detach(), P[i + 1].detach()) for i in range(0, len(P), 2)]}


def pose_rows(tr, q, tg):
    """Weighted log(T_target^-1 T_ee) of one configuration q [n] against tg [7]."""
    p, R = fk64(tr, q[None])[0]
    Rt = rot_of_quat(tg[3:])
    E, t = mm(Rt.T, R[0]), mv(Rt.T, p[0] - tg[:3])
    w = quat_of_rot(E)
    s = (w[1:].square().sum() + 1e-60).sqrt()
    th = 2 * torch.atan2(s, w[0])
    phi = th / s * w[1:]
    k = torch.where(th < 1e-3, 1 / 12 + th * th / 720, (1 - 0.5 * th * w[0] / s) / (th * th))
    a = torch.linalg.cross(phi, t)
    rho = t - 0.5 * a + k * torch.linalg.cross(phi, a)
    return torch.cat([TRAJ_COSTS["w_pos"] * rho, TRAJ_COSTS["w_rot"] * phi])


def exact_traj(c, seed):
    """LM over whole trajectories in float64 with dense normal equations.  Errors of converged
    endpoint poses are rounding residue and have no 64-bit value; nor have the counters."""
    if c["early_exit"]:
        return None          # stops at the first iterate within tolerance: decided by rounding at the edge
    tr, start, goal, init = traj_inputs(c, seed)
    parts = [exact_traj_batch(c, tr, start[:, b:b + 64], goal[:, b:b + 64], init[b:b + 64])
             for b in range(0, c["B"], 64)]
    return {"traj": torch.cat([p[0] for p in parts]), "cost": torch.cat([p[1] for p in parts]),
            "iters": None, "accepts": None, "status": None, "pos_err": None, "rot_err": None}


def exact_traj_batch(c, tr, start, goal, init):
    B, T, n = len(init), c["T"], c["n"]
    V, k, opt = T * n, TRAJ_COSTS, pk.Options()
    d64 = dict(dtype=torch.float64, device=DEV)
    lo, hi = (torch.as_tensor(x, **d64) for x in (tr.lower, tr.upper))
    D1 = torch.zeros((T - 1, T), **d64)
    i1 = torch.arange(T - 1, device=DEV)
    D1[i1, i1 + 1], D1[i1, i1] = 1.0, -1.0
    lin = [k["w_smooth"] * D1]
    for co, sc in (((-1 / 12, 16 / 12, -30 / 12, 16 / 12, -1 / 12), k["w_acc"] / k["dt"] ** 2),
                   ((-0.5, 1.0, 0.0, -1.0, 0.5), k["w_jerk"] / k["dt"] ** 3)):
        S = torch.zeros((T - 4, T), **d64)
        for o, v in enumerate(co):
            S[torch.arange(T - 4, device=DEV), torch.arange(T - 4, device=DEV) + o] = v * sc
        lin.append(S)
    Lm = torch.cat(lin)
    base = torch.kron((Lm.T @ Lm).contiguous(), torch.eye(n, **d64))
    st, gl = start.double().T.contiguous(), goal.double().T.contiguous()
    rows = torch.func.vmap(lambda q, t: pose_rows(tr, q, t))
    jac = torch.func.vmap(torch.func.jacfwd(lambda q, t: pose_rows(tr, q, t)))

    def parts(Q):
        lim = k["w_limit"] * ((Q - hi).clamp(min=0) + (lo - Q).clamp(min=0))
        dq = Q[:, 1:] - Q[:, :-1]
        vel = k["w_vel"] * (dq.abs() - VMAX * k["dt"]).clamp(min=0)
        sm = (Lm[None, :, :, None] * Q[:, None]).sum(2)
        return rows(Q[:, 0], st), rows(Q[:, -1], gl), lim, vel, sm

    def total(Q):
        return sum(x.flatten(1).square().sum(1) for x in parts(Q))

    Q = init.double()
    cost, lam = total(Q), torch.full((B,), opt.lambda0, **d64)
    for _ in range(c["iters"]):
        r0, r1, lim, vel, sm = parts(Q)
        J0, J1 = jac(Q[:, 0], st), jac(Q[:, -1], gl)
        A = base.expand(B, V, V).clone()
        A[:, :n, :n] += (J0[..., :, None] * J0[..., None, :]).sum(1)
        A[:, -n:, -n:] += (J1[..., :, None] * J1[..., None, :]).sum(1)
        dl = k["w_limit"] * ((Q > hi).double() - (Q < lo).double())
        sv = k["w_vel"] * torch.sign(Q[:, 1:] - Q[:, :-1]) * (vel > 0)
        g = dl * lim
        g[:, 1:] += sv * vel
        g[:, :-1] -= sv * vel
        g += (Lm[None, :, :, None] * sm[:, :, None]).sum(1)
        g[:, 0] += (J0 * r0[..., None]).sum(1)
        g[:, -1] += (J1 * r1[..., None]).sum(1)
        dg = dl.square()
        dg[:, 1:] += sv.square()
        dg[:, :-1] += sv.square()
        A.diagonal(dim1=1, dim2=2).add_(dg.flatten(1))
        off = A.diagonal(offset=n, dim1=1, dim2=2)
        off.sub_(sv.square().flatten(1))
        A.diagonal(offset=-n, dim1=1, dim2=2).sub_(sv.square().flatten(1))
        A.diagonal(dim1=1, dim2=2).add_(lam[:, None] * A.diagonal(dim1=1, dim2=2).clamp(min=opt.damping_floor))
        step = -torch.linalg.solve(A, g.flatten(1)[..., None])[..., 0]
        Qt = Q + step.unflatten(1, (T, n))
        ct = total(Qt)
        take = ct < cost
        Q, cost = torch.where(take[:, None, None], Qt, Q), torch.where(take, ct, cost)
        lam = torch.where(take, (lam / opt.nu_down).clamp(min=opt.lambda_min), (lam * opt.nu_up).clamp(max=opt.lambda_max))
    return Q, cost
