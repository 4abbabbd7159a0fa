"""Persistent launches of the star with fewer wavefronts than groups of 16
problems, as many, and more, and with a last group that is not full: every
problem is solved once, as in a plain launch."""
import numpy as np
import pytest

from tests.test_gpu_star import _problems, _solve, ctx  # noqa: F401  (ctx is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 16 * 256, 16 * 256 + 1, 16 * 700 + 15])
@pytest.mark.parametrize("k", [0, 3])
def test_star_persistent_grid(ctx, T, k):  # noqa: F811
    import torch

    import paper_2505_03728_amd as pk
    w, o = pk.Weights(w_pos=10.0, w_rest=0.01), pk.Options(max_iters=10, early_exit=True)
    rid, targets, seeds = _problems(ctx, T, 1, 17)
    g = {"rid": rid, "targets": targets, "seeds": seeds, "K": 1, "weights": w, "out": ctx.alloc_outputs(rid, T, 1)}
    # one wavefront per CU: 256 of them for up to 701 groups
    ctx.ik_solve_mixed([g], o, iters_per_launch=k, waves_per_cu=1, use_graph=False, mode=pk.SCHED_PER_GROUP)
    torch.cuda.synchronize()
    ref = _solve(ctx, rid, targets, seeds, 1, w, o)
    for key in ("joints", "cost", "iters", "accepts", "status", "pos_err", "iters_to_tol"):
        assert np.array_equal(g["out"][key].cpu().numpy(), ref[key], equal_nan=True), key
