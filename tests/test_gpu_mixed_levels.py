"""Mixed batches over every launch of a round: chains at both ends of each row
length of the path-pair kernel (8, 9, 13, 14 and 16 levels) and the per-lane
arm, one iteration range or several, every workgroup size.  The same
instantiations solve a group on its own, so the results are the same bits."""
import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import soa, targets_dev

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
AXES = "zyzyzyzyzyzyzyzy"


# (64: past the trees that one launch holds)
@pytest.mark.parametrize("scale", [1, 64])
@pytest.mark.parametrize("k,wg", [(0, 64), (4, 64), (0, 128), (5, 256)])
def test_mixed_levels_equal_separate(k, wg, scale):
    import paper_2505_03728_amd as pk
    import torch
    ctx = pk.Context(0)
    try:
        opt = pk.Options(max_iters=12, early_exit=True)
        groups, variants = [], []
        for i, (n, T, variant) in enumerate([(8, 33, pk.VARIANT_WAVE), (7, 130, pk.VARIANT_LANE),
                                             (16, 9, pk.VARIANT_WAVE), (9, 20, pk.VARIANT_WAVE),
                                             (13, 21, pk.VARIANT_WAVE), (14, 1, pk.VARIANT_WAVE)]):
            T *= scale
            tree = synth.chain(AXES[:n], 20 + i)
            rid = ctx.upload(tree)
            tg = oracle.targets_from(tree, synth.uniform_configs(tree, T, 50 + i))
            groups.append({"rid": rid, "targets": targets_dev(tree, tg, DEV), "K": 1,
                           "seeds": soa(synth.uniform_configs(tree, T, 60 + i), DEV),
                           "weights": pk.Weights(w_rest=0.01), "out": ctx.alloc_outputs(rid, T, 1)})
            variants.append(variant)
        ctx.ik_solve_mixed(groups, opt, iters_per_launch=k, use_graph=False, variants=variants,
                           workgroup_size=wg)
        for g, v in zip(groups, variants):
            o = pk.Options(max_iters=12, early_exit=True, variant=v)
            ref = ctx.ik_solve(g["rid"], g["targets"], g["seeds"], 1, g["weights"], o,
                               ctx.alloc_outputs(g["rid"], g["targets"].shape[1], 1))
            torch.cuda.synchronize()
            for key in ("joints", "cost", "iters", "accepts", "status", "pos_err", "rot_err"):
                a, b = g["out"][key].cpu().numpy(), ref[key].cpu().numpy()
                assert np.array_equal(a, b), (g["rid"], key)
    finally:
        ctx.close()
