"""Four lanes per problem against one lane per problem: single-chain batches
of up to 32768 problems (16384 from 9 joints) run on the first kernel, larger ones on the second,
and a problem's result does not depend on the batch it is in.  The same
problems are solved in a small batch and as the first ones of a large batch;
every output must agree bit for bit."""
import numpy as np
import pytest

import synth
from tests.gpu_util import soa

pytestmark = pytest.mark.gpu
BIG = 40000      # above the limits


def _robots():
    axes = "zyzyzyzyzy"
    out = {f"pose{n}": synth.chain(axes[:n], 40 + n) for n in range(2, 11)}
    for n in (2, 3, 5, 8):
        t = synth.chain(axes[:n], 60 + n)
        t.ee_kind = np.array([synth.EE_POSITION], np.int32)
        out[f"position{n}"] = t
    out["scara4"] = synth.scara4()
    out["mobile10"] = synth.mobile_arm7()
    return out


ROBOTS = _robots()


def _solve(pk, ctx, rid, targets, seeds, K, w, o, trace):
    import torch
    T = targets.shape[1]
    out = ctx.alloc_outputs(rid, T, K, best=True, trace_iters=trace)
    ctx.ik_solve(rid, targets, seeds, K, w, o, out)
    torch.cuda.synchronize()
    return {k: v for k, v in out.items() if not k.startswith("_")}


@pytest.mark.parametrize("name", list(ROBOTS))
@pytest.mark.parametrize("T,K,early", [(1, 1, True), (9, 8, True), (67, 3, False), (33, 64, True)])
def test_small_batches_equal_large(name, T, K, early):
    import torch

    import paper_2505_03728_amd as pk
    tree = ROBOTS[name]
    ctx = pk.Context(0)
    try:
        rid = ctx.upload(tree)
        pose = int(tree.ee_kind[0]) == synth.EE_POSE
        q = synth.uniform_configs(tree, T, 5)
        targets = ctx.fk(rid, soa(q, "cuda:0"))[0, :7 if pose else 3].contiguous()
        sd = synth.uniform_configs(tree, T * K, 6)
        sd[::11] *= 1.4                    # some seeds outside the limits
        seeds = soa(sd, "cuda:0")
        if T > 5:
            targets[1, 3] = float("nan")   # a target that is refused
            seeds[0, 2 * K] = float("inf")
        reps = BIG // (T * K) + 1
        big_t = targets.repeat(1, reps).contiguous()
        big_s = seeds.repeat(1, reps).contiguous()
        w = pk.Weights(w_rest=0.01)
        # a large pivot threshold sends some steps through the FP64 re-solve
        for o in (pk.Options(max_iters=25, early_exit=early),
                  pk.Options(max_iters=12, early_exit=early, pivot_rel=1e-3)):
            a = _solve(pk, ctx, rid, targets, seeds, K, w, o, 3)
            b = _solve(pk, ctx, rid, big_t, big_s, K, w, o, 3)
            N = T * K
            for k in a:
                n = a[k].shape[-1]
                x, y = a[k].view(torch.int32), b[k][..., :n].contiguous().view(torch.int32)
                assert n in (N, T)
                assert torch.equal(x, y), (name, k, int((x != y).sum()))
        if tree.dof >= 7 and T > 5:        # redundant: the rest term alone holds the last pivots
            assert int(((a["status"] & pk.FLAG_FP64) != 0).sum()) > 0
    finally:
        ctx.close()
