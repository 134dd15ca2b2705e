"""The range of knots in which a branch of seven bodies runs dID and the adjoint VJP one lane per body
on an MI355X: beyond two wavefronts of the quad layout per SIMD (8 knots per compute unit for dID, 16
for the VJP) and up to 54 knots per compute unit (2 wavefronts of 9 knots for each body beyond four),
both sides of both ends, with wavefronts that are not full, against the FP64 oracle at sampled knots, the
first and the last included. Outputs start as NaN; the tolerance is that of the parity tests (normwise
per knot, 1e-3)."""
import numpy as np
import pytest

from paper_2109_06976_amd import grid, synth
from paper_2109_06976_amd.build import prismatic_models

pytestmark = pytest.mark.gpu

ROBOTS = {"chain7": synth.chain7, "chain7-prism": lambda: prismatic_models()["chain7-prism"],
          "binary7": lambda: synth.random_model(np.array([-1, 0, 0, 1, 1, 2, 2], np.int32), 45)}


@pytest.mark.parametrize("per_cu, more", [(8, 0), (8, 1), (16, 1), (54, 0), (54, 1)])
@pytest.mark.parametrize("name", list(ROBOTS))
def test_derivatives_around_the_ends_of_the_range(orc, name, per_cu, more):
    import torch
    robot = ROBOTS[name]()
    n = robot.n
    N = per_cu * torch.cuda.get_device_properties(0).multi_processor_count + more
    m = grid.Model(robot)
    try:
        print(f"[gpu] dID, VJP {name} N={N}", flush=True)
        kn = synth.random_knots(n, N, 2500)
        g = synth.random_knots(n, N, 2501).qd
        q, qd, qdd, gb = (torch.from_numpy(a).cuda() for a in (kn.q, kn.qd, kn.tau, g))
        vec = [torch.full((N, n), float("nan"), device="cuda") for _ in range(3)]
        mat = [torch.full((N, n, n), float("nan"), device="cuda") for _ in range(2)]
        m.id_grad(q, qd, qdd, *mat)
        grid.fd_vjp_adjoint(m, q, qd, qdd, gb, *vec)
        torch.cuda.synchronize()
        for t in vec + mat:
            assert bool(torch.isfinite(t).all())
        idx = np.unique(np.concatenate([[0, N - 1], np.random.default_rng(12).integers(0, N, 40)]))
        it = torch.from_numpy(idx).cuda()
        der = [orc.rnea_grad(robot, kn.q[k], kn.qd[k], kn.tau[k]) for k in idx]
        t = np.stack([orc.minv_cholesky(robot, kn.q[k]) @ g[k].astype(np.float64) for k in idx])
        want = {"dq": np.stack([a for a, _ in der]), "dqd": np.stack([b for _, b in der]),
                "qbar": np.stack([-(a.T @ x) for (a, _), x in zip(der, t)]),
                "qdbar": np.stack([-(b.T @ x) for (_, b), x in zip(der, t)]), "taubar": t}
        for (key, ref), got in zip(want.items(), mat + vec):
            y = got[it].cpu().numpy().astype(np.float64)
            d, s = (np.abs(a).reshape(len(idx), -1).max(1) for a in (y - ref, ref))
            assert float((d / np.where(s > 0, s, 1.0)).max()) <= 1e-3, (name, N, key)
    finally:
        m.close()
