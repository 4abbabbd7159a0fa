"""Contexts of different threads share nothing: each thread creates, uses and
closes contexts of its own while the others do, with the plain results."""
import threading

import numpy as np
import pytest

import synth
from tests.gpu_util import soa

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
KEYS = ("joints", "cost", "iters", "status")


def test_contexts_of_four_threads():
    import torch

    import paper_2505_03728_amd as pk
    tree, T = synth.chain("zyzyzyz", 47), 300
    w, o = pk.Weights(w_rest=0.01), pk.Options(max_iters=6, early_exit=True)
    seeds = soa(synth.uniform_configs(tree, T, 6), DEV)
    ctx = pk.Context(0)
    rid = ctx.upload(tree)
    targets = ctx.fk(rid, soa(synth.uniform_configs(tree, T, 5), DEV))[0].contiguous()
    ref = ctx.ik_solve(rid, targets, seeds, 1, w, o, ctx.alloc_outputs(rid, T, 1))
    torch.cuda.synchronize()
    ref = {k: ref[k].cpu().numpy() for k in KEYS}
    bad = []

    def work(i):
        try:
            for _ in range(5):
                c = pk.Context(0)
                r = c.upload(tree)
                for k in (0, 2):
                    out = c.alloc_outputs(r, T, 1)
                    c.ik_solve_mixed([{"rid": r, "targets": targets, "seeds": seeds, "K": 1, "weights": w, "out": out}],
                                     o, iters_per_launch=k, waves_per_cu=4, use_graph=False)
                    torch.cuda.synchronize()
                    bad.extend((i, key) for key in KEYS
                               if not np.array_equal(out[key].cpu().numpy(), ref[key], equal_nan=True))
                c.close()
        except Exception as e:   # reported by the main thread
            bad.append((i, repr(e)))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    ctx.close()
    assert not bad
