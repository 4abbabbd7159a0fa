"""Device memory of a seeder's activations: at most what the buffers of its
passes take (per row: the input, the hidden layers and the output in BF16, a
BF16 gradient per layer the pass keeps, and for the layer-by-layer step FP32
pre-activations, one layer's FP32 gradient and the batch's joints)."""
import pytest

import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SLACK = 64 << 20      # allocation granularity, the code objects of a first launch


@pytest.mark.parametrize("hidden,depth,fused", [(512, 3, True), (384, 4, False)])
def test_activation_memory(hidden, depth, fused):
    import torch

    import paper_2505_03728_amd as pk
    tree = synth.chain("zyzyzyz", 47)
    ctx = pk.Context(0)
    try:
        rid = ctx.upload(tree)
        sd = pk.Seeder(ctx, rid, K=8, hidden=hidden, depth=depth)
        T = 1 << 18
        x = torch.zeros((128, 7), device=DEV)
        sd.grad(x, x.contiguous())
        tg = torch.zeros((7, T), device=DEV)
        tg[3] = 1.0
        seeds = torch.empty((7, T * 8), device=DEV)
        torch.cuda.synchronize()
        free0 = torch.cuda.mem_get_info()[0]
        sd.infer(tg, seeds)
        torch.cuda.synchronize()
        used = free0 - torch.cuda.mem_get_info()[0]
        row = 2 * 32 + 2 * hidden * depth + (2 + 4) * 64                    # X0, hidden, dY and Y
        row += 2 * hidden * (depth if fused else 1)                         # dZ in BF16
        if not fused:
            row += 4 * hidden * depth + 4 * hidden + 4 * 64 + 4 * 7         # Z, dZ, dY, Q
        # column-sum partials and losses: four rows per 128 of every layer, or one of a layer
        row += 4 * (4 * (depth * hidden + 64) / 128 + 1 if fused else hidden / 128 + 1 / 16)
        assert used <= T * row + SLACK, (used / T, row)
    finally:
        ctx.close()
