"""Batches of more threads than one grid can have (2^32) where a problem takes a
wavefront or a workgroup: the problems past the first launch's are solved too,
as the same problems in a small batch."""
import pytest

import synth
from tests.gpu_util import soa

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
W = 1 << 26           # wavefronts of 2^32 threads


@pytest.fixture()
def ctx():
    import torch

    import paper_2505_03728_amd as pk
    c = pk.Context(0)
    yield c
    c.close()
    torch.cuda.empty_cache()


def _same_tail(big, small, n):
    import torch
    torch.cuda.synchronize()
    assert torch.equal(big[..., :n], small[..., :n])
    assert torch.equal(big[..., -n:], small[..., -n:])


@pytest.mark.parametrize("variant", ["VARIANT_WAVE", "VARIANT_WAVE_JOINT"])
def test_wavefront_per_problem(ctx, variant):
    import torch

    import paper_2505_03728_amd as pk
    tree, N, n = synth.chain("zyz", 43), W + 100, 200
    rid = ctx.upload(tree)
    targets = ctx.fk(rid, soa(synth.uniform_configs(tree, 1, 5), DEV))[0].contiguous()
    some = soa(synth.uniform_configs(tree, 2 * n, 6), DEV)
    seeds = torch.zeros((3, N), device=DEV)
    seeds[:, :n], seeds[:, -n:] = some[:, :n], some[:, n:]
    w, o = pk.Weights(w_rest=0.01), pk.Options(max_iters=1, variant=getattr(pk, variant))
    big = ctx.ik_solve(rid, targets, seeds, N, w, o, ctx.alloc_outputs(rid, 1, N, full=False))
    small = ctx.ik_solve(rid, targets, some, 2 * n, w, o, ctx.alloc_outputs(rid, 1, 2 * n, full=False))
    _same_tail(big["joints"], small["joints"], n)


def test_beam(ctx):
    import torch

    import paper_2505_03728_amd as pk
    tree, T, n = synth.chain("zy", 42), W + 100, 200
    rid = ctx.upload(tree)
    q, s = (soa(synth.uniform_configs(tree, 2 * n, i), DEV) for i in (5, 6))
    few = ctx.fk(rid, q)[0].contiguous()
    fill = lambda a: torch.cat([a[:, :n], a[:, :1].expand(-1, T - 2 * n), a[:, n:]], 1).contiguous()
    w, o = pk.Weights(w_rest=0.01), pk.Options(max_iters=1)
    args = dict(n_seeds=1, iters0=1, keep=1, iters1=1)
    big = ctx.ik_beam(rid, fill(few), fill(s), w, o, **args)
    small = ctx.ik_beam(rid, few, s, w, o, **args)
    _same_tail(big["best_joints"], small["best_joints"], n)
    _same_tail(big["cost"], small["cost"], n)


def test_trajectories(ctx):
    import torch

    import paper_2505_03728_amd as pk
    tree, T, n = synth.scara4(), 5, 100
    B = (1 << 24) + 50
    rid = ctx.upload(tree)
    qa, qb = (soa(synth.uniform_configs(tree, 2 * n, i), DEV) for i in (41, 42))
    st, gl = (ctx.fk(rid, q)[0].contiguous() for q in (qa, qb))
    s = torch.linspace(0, 1, T, device=DEV)[None, :, None]
    init = ((1 - s) * qa.T[:, None] + s * qb.T[:, None]).contiguous()
    wide = lambda a: torch.cat([a[:, :n], a[:, :1].expand(-1, B - 2 * n), a[:, n:]], 1).contiguous()
    costs = {"dt": 0.05, "w_pos": 10.0, "w_rot": 5.0, "w_limit": 10.0, "w_smooth": 0.1, "w_vel": 0.0,
             "w_acc": 0.05, "w_jerk": 0.01}
    many = torch.cat([init[:n], init[:1].expand(B - 2 * n, -1, -1), init[n:]]).contiguous()
    o = pk.Options(max_iters=0)
    big = ctx.traj_solve(rid, wide(st), wide(gl), many, costs, o)
    small = ctx.traj_solve(rid, st, gl, init, costs, o)
    _same_tail(big["cost"], small["cost"], n)
    _same_tail(big["pos_err"], small["pos_err"], n)
