"""The scheduler keeps a batch's description and graphs by what the call
passes: a call that differs in one number's last bits, or in a group's lanes per
problem, is not the one before it."""
import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import soa, targets_dev
from tests.test_gpu_wave import _hand5

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
KEYS = ("joints", "cost", "iters", "status")


@pytest.fixture(scope="module")
def ctx():
    import paper_2505_03728_amd as pk
    c = pk.Context(0)
    yield c
    c.close()


def _problems(ctx, tree, T):
    rid = ctx.upload(tree)
    tg = oracle.targets_from(tree, synth.uniform_configs(tree, T, 5))
    return rid, targets_dev(tree, tg, DEV), soa(synth.uniform_configs(tree, T, 6), DEV)


def _host(out):
    return {k: out[k].cpu().numpy() for k in KEYS}


def _plain(ctx, rid, targets, seeds, w, o):
    import torch
    out = ctx.ik_solve(rid, targets, seeds, 1, w, o, ctx.alloc_outputs(rid, targets.shape[1], 1))
    torch.cuda.synchronize()
    return _host(out)


@pytest.mark.parametrize("mode,graph", [(0, False), (0, True), (1, True)])
@pytest.mark.parametrize("name", ["w_pos", "lambda0"])
def test_numbers_by_their_bits(ctx, mode, graph, name):
    import torch

    import paper_2505_03728_amd as pk
    rid, targets, seeds = _problems(ctx, synth.chain("zyzyzyz", 47), 200)
    out = ctx.alloc_outputs(rid, 200, 1)
    refs = []
    for x in (1.0, 1.0 + 2.0 ** -20):
        w = pk.Weights(w_pos=x if name == "w_pos" else 1.0, w_rest=0.01)
        o = pk.Options(max_iters=6, lambda0=x if name == "lambda0" else 1.0)
        refs.append(_plain(ctx, rid, targets, seeds, w, o))
        ctx.ik_solve_mixed([{"rid": rid, "targets": targets, "seeds": seeds, "K": 1, "weights": w, "out": out}], o,
                           waves_per_cu=4, use_graph=graph, mode=mode)
        torch.cuda.synchronize()
        got = _host(out)
        for k in KEYS:
            assert np.array_equal(got[k], refs[-1][k], equal_nan=True), (x, k)
    assert not np.array_equal(refs[0]["cost"], refs[1]["cost"])


def test_lanes_per_problem(ctx):
    import torch

    import paper_2505_03728_amd as pk
    rid, targets, seeds = _problems(ctx, _hand5(), 64)
    out = ctx.alloc_outputs(rid, 64, 1)
    w, refs = pk.Weights(w_pos=10.0, w_rest=0.01), []
    for variant in (pk.VARIANT_WAVE, pk.VARIANT_WAVE_JOINT):
        refs.append(_plain(ctx, rid, targets, seeds, w, pk.Options(max_iters=6, variant=variant)))
        ctx.ik_solve_mixed([{"rid": rid, "targets": targets, "seeds": seeds, "K": 1, "weights": w, "out": out}],
                           pk.Options(max_iters=6), waves_per_cu=4, variants=[variant], mode=pk.SCHED_PER_GROUP)
        torch.cuda.synchronize()
        got = _host(out)
        for k in KEYS:
            assert np.array_equal(got[k], refs[-1][k], equal_nan=True), (variant, k)
    assert not np.array_equal(refs[0]["joints"], refs[1]["joints"])
