"""The trajectory solver at its largest number of variables (T n = 256, scara of
4 joints), where the band solve's reads past the last row, clamped rows and a
full last chunk of the backward solve meet, and around it.

The trajectory after two iterations against the FP64 oracle's, within 1e-5 rad
or m (FP32 kinematics part from the oracle by about 1e-6, see
test_gpu_traj_shapes; a wrong row of the solve moves its variable by about a
step, 1e-2 and more).  The cost the solver reports is checked against the FP64
cost of the trajectory it returns, within what FP32 arithmetic can do: six
roundings (u = 2^-24) of a stencil row's terms, whose weights divided by dt^2 and
dt^3 are large here, and the pose rows' FP32 errors."""
import numpy as np
import pytest

import synth
from oracle import traj

from .gpu_util import FP32_RES_ERR
from .test_gpu_traj import _run, ctx  # noqa: F401  (ctx is a fixture)

pytestmark = pytest.mark.gpu

STENCIL = {"w_acc": (2, np.array([1, 16, 30, 16, 1]) / 12), "w_jerk": (3, np.array([0.5, 1, 0, 1, 0.5]))}


@pytest.mark.parametrize("T", [62, 63, 64])
def test_traj_longest(ctx, T):  # noqa: F811
    tree, n, B = synth.scara4(), 4, 8
    qa = synth.uniform_configs(tree, B, 41)
    qb = np.clip(qa + 0.4 * np.random.default_rng(42).standard_normal(qa.shape),
                 np.asarray(tree.lower)[tree.var_joints], np.asarray(tree.upper)[tree.var_joints])
    s = np.linspace(0, 1, T)[None, :, None]
    init = synth.f32((1 - s) * qa[:, None] + s * qb[:, None] +
                     0.05 * np.sin(np.pi * s) * np.ones((1, 1, n)))
    costs = {"T": T, "dt": 0.05, "w_pos": 10.0, "w_rot": 5.0, "w_limit": 10.0, "w_smooth": 0.1,
             "w_vel": 1.0, "vmax": [2.0] * n, "w_acc": 0.05, "w_jerk": 0.01}
    o = dict(synth.workload("traj", targets=1)["options"], max_iters=2)
    res, st, gl = _run(ctx, tree, qa, qb, init, costs, o)
    u = 2.0 ** -24
    for b in range(B):
        ora = traj.lm_solve(tree, st[b], gl[b], costs, o, init[b].astype(np.float64))
        q = res["traj"][b].astype(np.float64)
        assert np.isfinite(q).all() and res["status"][b] == ora["status"]
        assert np.abs(q - ora["Q"]).max() <= 1e-5, (b, np.abs(q - ora["Q"]).max())
        e2 = 6 * FP32_RES_ERR ** 2 * (costs["w_pos"] ** 2 + costs["w_rot"] ** 2)   # (both ends, 3 rows each)
        for w, (p, c) in STENCIL.items():
            rows = sum(c[i] * np.abs(q[i:T - 4 + i]) for i in range(5)) * costs[w] / costs["dt"] ** p
            e2 += ((6 * u * rows) ** 2).sum()
        c64 = traj.cost(tree, st[b], gl[b], costs, q)
        bound = 2 * np.sqrt(c64 * e2) + e2 + 300 * u * c64
        print(f"T={T} {b}: cost {c64:.3e}, off by {abs(res['cost'][b] - c64):.1e}, bound {bound:.1e}")
        assert abs(res["cost"][b] - c64) <= bound, b
