"""A seeder call that is only recorded into a graph leaves the weights' copies in
fragment order as they were: the next inference builds them, and a replay
gives the eager values."""
import numpy as np
import pytest

import synth
from tests.gpu_util import soa

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("call", ["grad", "forward"])
def test_recorded_call_builds_nothing(call):
    import torch

    import paper_2505_03728_amd as pk
    rng = np.random.default_rng(3)
    sizes = [7, 256, 256, 56]
    init = [(rng.uniform(-1, 1, (o, i)).astype(np.float32) / np.float32(np.sqrt(i)),
             rng.uniform(-1, 1, o).astype(np.float32)) for i, o in zip(sizes[:-1], sizes[1:])]
    tree = synth.chain("zyzyzyz", 47)
    ctx = pk.Context(0)
    try:
        rid = ctx.upload(tree)
        sd = pk.Seeder(ctx, rid, K=8, hidden=256, depth=2, init=init)
        B = 256
        x = torch.from_numpy(rng.standard_normal((B, 7)).astype(np.float32)).to(DEV)
        q = soa(synth.uniform_configs(tree, B, 5), DEV).T.contiguous()
        want = sd.forward(x, layers=True).clone()     # also sizes the activations; no fragment copies
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            res = sd.grad(x, q) if call == "grad" else sd.forward(x)
        assert torch.equal(sd.forward(x), want)       # recorded, never run
        for _ in range(3):
            res.zero_()
            graph.replay()
            torch.cuda.synchronize()
            eager = sd.grad(x, q) if call == "grad" else want
            assert torch.equal(res, eager)
            assert torch.equal(sd.forward(x), want)
    finally:
        ctx.close()
