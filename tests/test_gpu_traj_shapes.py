"""Trajectory solver where its band solve can go wrong: every chain size at
the shortest trajectory (T = 5), one step around a whole number of the
factorisation's column blocks, and the most variables (T n <= 256), so the last
block is full, nearly empty or the only one.

Two iterations of 8 trajectories against the FP64 oracle with the limits of
test_gpu_traj (1e-3 in cost, relative, and in radians): over two iterations
FP32 kinematics part from the oracle by about 1e-6.
"""
import numpy as np
import pytest

import synth
from .test_gpu_traj import _compare, _run, ctx  # noqa: F401  (ctx is a fixture)

pytestmark = pytest.mark.gpu

TREES = {4: lambda: synth.scara4(), 6: lambda: synth.chain("zyzyzy", 4, name="chain6"),
         7: lambda: synth.workload("traj", targets=1)["tree"], 10: lambda: synth.mobile_arm7(0)}


# The cost of a 64-step prismatic chain is nearly all five-point stencils: the
# FP32 residuals' rounding is multiplied by up to 30 / (12 dt^2), which leaves
# about 1e-6 rad of roughness in the solved trajectory and up to 2.1e-3 of a
# cost of 9e-4 (measured), above the limit that the other shapes keep.
LONG = pytest.param(4, 64, marks=pytest.mark.xfail(
    reason="FP32 residual rounding through the stencils is above 1e-3 of this small cost"))


@pytest.mark.parametrize("n,T", [(4, 5), (4, 13), LONG, (6, 5), (6, 11), (6, 42), (7, 5),
                                 (7, 9), (7, 10), (7, 36), (10, 5), (10, 13), (10, 25)])
def test_traj_shapes(ctx, n, T):  # noqa: F811
    tree = TREES[n]()
    B = 8
    qa = synth.uniform_configs(tree, B, 41)
    qb = np.clip(qa + 0.4 * np.random.default_rng(42).standard_normal(qa.shape),
                 np.asarray(tree.lower)[tree.var_joints], np.asarray(tree.upper)[tree.var_joints])
    s = np.linspace(0, 1, T)[None, :, None]
    init = synth.f32((1 - s) * qa[:, None] + s * qb[:, None] +
                     0.05 * np.sin(np.pi * s) * np.ones((1, 1, n)))
    costs = {"T": T, "dt": 0.05, "w_pos": 10.0, "w_rot": 5.0, "w_limit": 10.0, "w_smooth": 0.1,
             "w_vel": 1.0, "vmax": [2.0] * n, "w_acc": 0.05, "w_jerk": 0.01}
    o = dict(synth.workload("traj", targets=1)["options"], max_iters=2)
    _compare(tree, *_run(ctx, tree, qa, qb, init, costs, o), init, costs, o, f"n={n} T={T}")
