"""Single-chain batches around the line between four lanes and one lane per
problem: best-of-K in the launch just below it, in a launch of its own just
above it, and the line of 8 joints with and without the rest term.  The same
problems as the first ones of a batch above every line give the same bits, the
best-of-K outputs included."""
import pytest

import synth
from tests.gpu_util import soa

pytestmark = pytest.mark.gpu

KEYS = ("joints", "cost", "iters", "status", "best_index", "best_joints", "target_success")


@pytest.mark.parametrize("n,T,K,w_rest", [(7, 10752, 3, 0.01), (7, 10753, 3, 0.01), (7, 512, 33, 0.01),
                                          (7, 513, 33, 0.01), (8, 16400, 1, 0.01), (8, 16400, 1, 0.0)])
def test_batches_at_the_line(n, T, K, w_rest):
    import torch

    import paper_2505_03728_amd as pk
    tree = synth.chain("zyzyzyzy"[:n], 40 + n)
    ctx = pk.Context(0)
    try:
        rid = ctx.upload(tree)
        q = synth.uniform_configs(tree, T, 5)
        targets = ctx.fk(rid, soa(q, "cuda:0"))[0].contiguous()
        seeds = soa(synth.uniform_configs(tree, T * K, 6), "cuda:0")
        w, o = pk.Weights(w_rest=w_rest), pk.Options(max_iters=6, early_exit=True)
        reps = 66000 // (T * K) + 1
        a = ctx.ik_solve(rid, targets, seeds, K, w, o, ctx.alloc_outputs(rid, T, K, best=True))
        b = ctx.ik_solve(rid, targets.repeat(1, reps).contiguous(), seeds.repeat(1, reps).contiguous(), K, w, o,
                         ctx.alloc_outputs(rid, T * reps, K, best=True))
        torch.cuda.synchronize()
        for k in KEYS:
            x = a[k].view(torch.int32)
            y = b[k][..., :x.shape[-1]].contiguous().view(torch.int32)
            assert torch.equal(x, y), (k, int((x != y).sum()))
    finally:
        ctx.close()
