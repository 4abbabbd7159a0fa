"""The three-launch training step over the shapes it serves (hidden widths 128,
256 and 512, one to three hidden layers) and one it leaves to the layer-by-layer
pass: loss and gradients against the BF16-emulation oracle at the sizes where
the row split differs (one slice, an odd number of 32-row steps per slice, more
slices than wavefronts), and the weight copies the inference pass reads after a
step.  Tolerances are those of the gradient parity test (2e-2 relative per
tensor, 5e-2 of the RMS per element, loss to 1e-3)."""
import numpy as np
import pytest

import synth
from oracle import mlp
from tests.test_gpu_seeder import _dev, _inputs, _max_over_rms, _rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,depth,K,B", [(128, 1, 8, 128), (128, 3, 3, 1152), (256, 1, 8, 640),
                                              (256, 3, 2, 384), (512, 1, 8, 128), (512, 2, 8, 1152),
                                              (512, 3, 1, 4224), (128, 4, 8, 256)])
def test_step_gradients_and_weight_copies(hidden, depth, K, B):
    import torch

    import paper_2505_03728_amd as pk
    ctx = pk.Context(0)
    try:
        rid = ctx.upload(synth.arm7(0))
        init = synth.mlp_init([7] + [hidden] * depth + [7 * K], 90 + depth)
        sd = pk.Seeder(ctx, rid, K=K, hidden=hidden, depth=depth, init=init)
        x, q = _inputs(B, 8)
        loss = sd.grad(_dev(x), _dev(q))
        torch.cuda.synchronize()
        g = sd.get(1)
        y, cache = mlp.forward(init, x, emulate_bf16=True)
        lo, _, dy = mlp.min_over_k_loss(y, q, K)
        go = mlp.backward(init, cache, dy, emulate_bf16=True)
        assert abs(loss.item() - lo) <= 1e-3 * lo
        for li, ((gW, gb), (oW, ob)) in enumerate(zip(g, go)):
            assert _rel(gW, oW) <= 2e-2 and _rel(gb, ob) <= 2e-2, li
            assert _max_over_rms(gW, oW) <= 5e-2 and _max_over_rms(gb, ob) <= 5e-2, li
        # a step, in the order of a permutation: the inference pass then reads the new weights
        perm = synth.epoch_permutation(B, 4, 0)[None]
        log = torch.zeros(1, device="cuda:0")
        sd.train(_dev(q.T), batch=B, epochs=1, lr=1e-2, perm=torch.from_numpy(perm).cuda(), loss_log=log)
        xd = _dev(x)
        yf, yl = sd.forward(xd), sd.forward(xd, layers=True)
        torch.cuda.synchronize()
        assert torch.equal(yf, yl)
        assert abs(log.item() - lo) <= 1e-3 * lo
        yo, _ = mlp.forward(sd.get(0), x, emulate_bf16=True)
        assert _rel(yf.cpu().numpy(), yo) <= 1e-3
        assert not np.array_equal(sd.get(0)[0][0], init[0][0].astype(np.float32))
    finally:
        ctx.close()
