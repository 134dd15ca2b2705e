"""One lane per body on trees of segments (a segment is a run of bodies with one child each):
sums by doubling within segments of up to 17 bodies and across branch points at two depths,
and rows of a group of branches that are not adjacent in the robot, against the FP64 oracle at
knot counts around a wavefront's. The tolerances are those of the parity tests (normwise per
knot: vectors 1e-4, matrices 1e-3).
"""
import numpy as np
import pytest

from paper_2109_06976_amd import grid, synth
from paper_2109_06976_amd.build import tree_models

pytestmark = pytest.mark.gpu

TOL = {"qdd": 1e-4, "Minv": 1e-3, "dqdd_dq": 1e-3, "dqdd_dqd": 1e-3}


@pytest.mark.parametrize("name, knots", [("chain17", 3), ("branches13", 7), ("pairs8", 16)])
def test_team_gradient_on_trees_of_segments(orc, name, knots):
    import torch
    robot = tree_models()[name]
    n = robot.n
    m = grid.Model(robot)
    try:
        grid.tune_apply(m, {1 << 22: grid.BUILD_LANE})
        for N in (1, knots, 2 * knots + 1):
            print(f"[gpu] team trees {name} N={N}", flush=True)
            kn = synth.random_knots(n, N, 1600 + N)
            ins = [torch.from_numpy(a).cuda() for a in (kn.q, kn.qd, kn.tau)]
            outs = [torch.full((N, n) + (n,) * (k > 0), float("nan"), device="cuda")
                    for k in range(4)]
            m.fd_grad(*ins, *outs, N=N)
            torch.cuda.synchronize()
            ref = orc.fd_grad_batch(robot, kn.q, kn.qd, kn.tau)
            for (key, tol), out in zip(TOL.items(), outs):
                d = np.abs(out.cpu().numpy().astype(np.float64) - ref[key]).reshape(N, -1).max(1)
                s = np.abs(ref[key]).reshape(N, -1).max(1)
                err = float((d / np.where(s > 0, s, 1.0)).max())
                assert err <= tol, (name, N, key, err)
    finally:
        m.close()
