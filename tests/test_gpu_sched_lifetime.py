"""Graphs that leave the scheduler's cache, and the context itself, while their
replays are queued: more schedules than the cache holds, one after the other
without a wait, and the context closed behind them.  Every output is that of
a plain solve."""
import numpy as np
import pytest

import synth
from tests.gpu_util import soa

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
KEYS = ("joints", "cost", "iters", "status")


def test_graphs_leave_the_cache_in_flight():
    import torch

    import paper_2505_03728_amd as pk
    tree, T = synth.chain("zyzyzyz", 47), 2000
    w, o = pk.Weights(w_rest=0.01), pk.Options(max_iters=20, early_exit=True)
    q = synth.uniform_configs(tree, T, 5)
    seeds = soa(synth.uniform_configs(tree, T, 6), DEV)
    ctx = pk.Context(0)
    rid = ctx.upload(tree)
    targets = ctx.fk(rid, soa(q, DEV))[0].contiguous()
    ref = ctx.ik_solve(rid, targets, seeds, 1, w, o, ctx.alloc_outputs(rid, T, 1))
    outs = [ctx.alloc_outputs(rid, T, 1) for _ in range(3)]
    torch.cuda.synchronize()
    for k in range(1, 21):              # 20 schedules x 3 batches: 60 graphs, 16 held
        for out in outs:
            ctx.ik_solve_mixed([{"rid": rid, "targets": targets, "seeds": seeds, "K": 1, "weights": w, "out": out}],
                               o, iters_per_launch=k, waves_per_cu=4)
    ctx.close()
    torch.cuda.synchronize()
    for out in outs:
        for key in KEYS:
            assert np.array_equal(out[key].cpu().numpy(), ref[key].cpu().numpy(), equal_nan=True), key
