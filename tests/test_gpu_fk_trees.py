"""Forward kinematics over tree shapes: the kernel keeps the running frame in
registers and the frames later branches start from in LDS slots, so the shapes
cover no slot, one, nested ones and as many as a robot can need at once.

Tolerances: those of the FK parity test (1e-5 m, 1e-5 on rotation entries),
scaled with the depth of the tree relative to its 13 levels where deeper."""
import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import quat_to_R, soa

pytestmark = pytest.mark.gpu


def _tree(parent, ees, seed, types=None):
    rng = np.random.default_rng(seed)
    n = len(parent)
    h = rng.normal(size=(n, 4))
    kinds = [k % 2 for k in range(len(ees))]
    return synth._finish("t", parent, h / np.linalg.norm(h, axis=1, keepdims=True),
                         rng.uniform(-0.1, 0.1, (n, 3)), [synth._AX["xyz"[j % 3]] for j in range(n)],
                         rng.uniform(0.5, 3.0, n), ees, rng.uniform(-0.1, 0.1, (len(ees), 3)),
                         np.tile([1.0, 0, 0, 0], (len(ees), 1)), kinds, joint_type=types)


SHAPES = {
    "chain": (list(range(-1, 11)), [11, 4]),
    "star_breadth_first": ([-1] * 32 + list(range(32)), list(range(56, 64))),     # 32 live frames
    "binary": ([-1] + [(j - 1) // 2 for j in range(1, 63)], [62, 31, 40, 55, 0]),
    "nested_depth_first": ([-1, 0, 1, 2, 2, 1, 5, 5, 0, 8, 8, -1, 11], [3, 4, 6, 7, 9, 10, 12]),
    "one_joint": ([-1], [0]),
}


@pytest.mark.parametrize("N", [1, 63, 65, 200])
@pytest.mark.parametrize("name", list(SHAPES))
def test_fk_tree_shapes(name, N):
    import torch

    import paper_2505_03728_amd as pk
    parent, ees = SHAPES[name]
    types = [1 if j % 5 == 3 else 0 for j in range(len(parent))]
    tree = _tree(parent, ees, 7, types)
    ctx = pk.Context(0)
    try:
        rid = ctx.upload(tree)
        q = synth.uniform_configs(tree, N, 3)
        ee, fr = ctx.fk(rid, soa(q, "cuda:0"), frames=True)
        ee_only = ctx.fk(rid, soa(q, "cuda:0"))
        torch.cuda.synchronize()
        assert torch.equal(ee, ee_only)
        ee, fr = ee.cpu().numpy().astype(np.float64), fr.cpu().numpy().astype(np.float64)
    finally:
        ctx.close()
    worst = 0.0
    for p in sorted({0, N // 2, N - 1}):
        R, pos, Re, pe = oracle.fk(tree, q[p])
        for k in range(tree.m):
            assert ee[k, 3, p] >= 0
            worst = max(worst, np.abs(ee[k, :3, p] - pe[k]).max(),
                        np.abs(quat_to_R(ee[k, 3:, p]) - Re[k]).max())
        for j in range(tree.n):
            worst = max(worst, np.abs(fr[j, 9:, p] - pos[j]).max(),
                        np.abs(fr[j, :9, p].reshape(3, 3) - R[j]).max())
    assert worst <= 1e-5, worst
