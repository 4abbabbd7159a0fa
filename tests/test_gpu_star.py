"""The star's four lanes per problem against the per-lane kernel, which serves
target_exit: with one seed per target there is no other problem to end on, so
the two kernels are asked for the same thing and give the same bits (the
results, flags and traces), non-finite problems included.  Best-of-K in the
launch, and the resumable launches of a mixed batch, against the plain results."""
import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import soa, targets_dev
from tests.test_gpu_selection import _pick

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def ctx():
    import paper_2505_03728_amd as pk
    c = pk.Context(0)
    yield c
    c.close()


def _problems(ctx, T, K, seed):
    tree = synth.workload("mixed84k", scale=0.001)["groups"][1]["tree"]
    assert tree.dof == 16
    rid = ctx.upload(tree)
    tg = oracle.targets_from(tree, synth.uniform_configs(tree, T, seed))
    seeds = synth.uniform_configs(tree, T * K, seed + 1)
    seeds[::97, 9] = np.nan
    return rid, targets_dev(tree, tg, DEV), soa(seeds, DEV)


def _solve(ctx, rid, targets, seeds, K, w, o, **kw):
    import torch
    out = ctx.ik_solve(rid, targets, seeds, K, w, o, ctx.alloc_outputs(rid, targets.shape[1], K, **kw))
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in out.items() if hasattr(v, "cpu")}


@pytest.mark.parametrize("T", [1, 16, 63, 65, 1000])
@pytest.mark.parametrize("w_rest", [0.01, 0.0])
def test_star_equals_per_lane(ctx, T, w_rest):
    import paper_2505_03728_amd as pk
    rid, targets, seeds = _problems(ctx, T, 1, 5)
    w = pk.Weights(w_pos=10.0, w_rest=w_rest)
    a, b = (_solve(ctx, rid, targets, seeds, 1, w,
                   pk.Options(max_iters=25, early_exit=True, target_exit=x), trace_iters=25)
            for x in (False, True))
    for k in a:
        assert np.array_equal(a[k], b[k], equal_nan=True), k


@pytest.mark.parametrize("T,K", [(30, 5), (3, 64), (2, 70)])
def test_star_best_of_k(ctx, T, K):
    import paper_2505_03728_amd as pk
    rid, targets, seeds = _problems(ctx, T, K, 7)
    r = _solve(ctx, rid, targets, seeds, K, pk.Weights(w_pos=10.0, w_rest=0.01),
               pk.Options(max_iters=8, early_exit=True), best=True)
    for t in range(T):
        s = slice(t * K, (t + 1) * K)
        b, any_ = _pick(r["status"][s], r["cost"][s], r["pose_cost"][s])
        assert r["best_index"][t] == b and r["target_success"][t] == int(any_)
        assert np.array_equal(r["best_joints"][:, t], r["joints"][:, t * K + b], equal_nan=True)


@pytest.mark.parametrize("k", [0, 4])
def test_star_in_mixed_batches(ctx, k):
    import paper_2505_03728_amd as pk
    import torch
    w, o = pk.Weights(w_pos=10.0, w_rest=0.01), pk.Options(max_iters=20, early_exit=True)
    for mode in (pk.SCHED_SINGLE, pk.SCHED_PER_GROUP):
        groups = []
        for T, seed in ((33, 11), (1000, 13)):
            rid, targets, seeds = _problems(ctx, T, 1, seed)
            groups.append({"rid": rid, "targets": targets, "seeds": seeds, "K": 1, "weights": w,
                           "out": ctx.alloc_outputs(rid, T, 1)})
        ctx.ik_solve_mixed(groups, o, iters_per_launch=k, use_graph=False, mode=mode)
        torch.cuda.synchronize()
        for g in groups:
            ref = _solve(ctx, g["rid"], g["targets"], g["seeds"], 1, w, o)
            for key in ("joints", "cost", "iters", "accepts", "status", "pos_err", "iters_to_tol"):
                assert np.array_equal(g["out"][key].cpu().numpy(), ref[key], equal_nan=True), (mode, key)
