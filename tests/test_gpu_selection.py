"""The kernels that list, rank and pick results by whole wavefronts, where they
can go wrong: fewer and more candidates than lanes, targets that are not a whole
number of wavefronts or blocks, several fallback stages, and non-finite
candidates.  Selections are compared exactly: the beam's with the oracle's on
the GPU's own values, the pipeline's with its rule applied to a separate solve of
the same problems (which gives the same bits)."""
import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import soa, targets_dev
from tests.test_gpu_beam import _case, _check_selection, _run

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def ctx():
    import paper_2505_03728_amd as pk
    c = pk.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("T,K,keep", [(1, 1, 1), (3, 5, 5), (5, 33, 10), (9, 63, 1), (6, 64, 64)])
def test_beam_selection(ctx, T, K, keep):
    tree, tg, seeds, wl = _case(T)
    seeds = seeds.reshape(T, 64, -1)[:, :K].reshape(T * K, -1).copy()
    seeds[::7] = np.nan                      # ranks after every number, and all seeds of (1, 1)
    sch = {"n_seeds": K, "iters0": 6, "keep": keep, "iters1": 10}
    o = dict(wl["options"], early_exit=True)
    _check_selection(_run(ctx, ctx.upload(tree), tree, tg, seeds, wl["weights"], o, sch), T, sch)


def _pick(status, cost, pcost):
    """Lowest cost of the converged, else lowest pose cost; `<` from the first on."""
    conv = (status & 0xFF) == 0
    v = cost if conv.any() else pcost
    b = -1
    for k in range(len(v)):
        if conv.any() and not conv[k]:
            continue
        if b < 0 or v[k] < v[b]:
            b = k
    return b, bool(conv.any())


@pytest.mark.parametrize("T,Kf,chunk", [(1, 1, 0), (9, 70, 0), (130, 130, 65), (1030, 24, 7), (2049, 3, 1)])
def test_seeded_fallback_selection(ctx, T, Kf, chunk):
    import paper_2505_03728_amd as pk
    import torch
    tree = synth.arm7(0)
    rid = ctx.upload(tree)
    tg = oracle.targets_from(tree, synth.uniform_configs(tree, T, 71))
    targets = targets_dev(tree, tg, DEV)
    fb = synth.uniform_configs(tree, T * Kf, 72)
    fb[::5 * Kf] = np.nan                    # every fifth target's first seed
    seeds = soa(fb, DEV)
    sd = pk.Seeder(ctx, rid, K=8, hidden=128, depth=1)
    w, o = pk.Weights(w_rest=0.01), pk.Options(max_iters=14, early_exit=True)
    res = ctx.ik_solve_seeded(rid, targets, sd, w, pk.Options(max_iters=1, early_exit=True), fallback=o,
                              fallback_seeds=seeds, fallback_K=Kf, fallback_chunk=chunk, counters=True)
    sep = ctx.ik_solve(rid, targets, seeds, Kf, w, o, ctx.alloc_outputs(rid, T, Kf))
    torch.cuda.synchronize()
    res = {k: v.cpu().numpy() for k, v in res.items()}
    sep = {k: v.cpu().numpy() for k, v in sep.items() if hasattr(v, "cpu")}
    rows = {k: sep[k].reshape(T, Kf) for k in ("status", "cost", "pose_cost", "iters_to_tol")}
    c = chunk or Kf
    todo = np.nonzero(res["source"] != 0)[0]
    ran = 0
    for t in todo:
        kr = Kf
        for c1 in range(c, Kf, c):           # stages up to the first with a converged problem
            if ((rows["status"][t, c1 - c:c1] & 0xFF) == 0).any():
                kr = c1
                break
        ran += kr
        b, any_ = _pick(rows["status"][t, :kr], rows["cost"][t, :kr], rows["pose_cost"][t, :kr])
        itt = rows["iters_to_tol"][t, :kr]
        assert res["source"][t] == (1 if any_ else -1)
        assert res["target_success"][t] == int(any_)
        assert res["iters_to_tol"][t] == (itt[itt >= 0].min() if any_ else -1)
        np.testing.assert_array_equal(res["best_joints"][:, t], sep["joints"][:, t * Kf + b])
    assert res["n_fallback"][0] == len(todo) and res["n_fallback_problems"][0] == ran
    assert len(todo) > T // 2                # the refinement of an untrained net solves few
