"""Branches of five bodies on an MI355X run dFD, dID and the adjoint VJP one lane per body up to
two wavefronts per compute unit, one lane per problem beyond: both sides of that end against the FP64
oracle at sampled knots, the first and the last included (outputs start as NaN; normwise per knot,
1e-3, the tolerance of the parity tests), and the 2-norm errors of dFD over 2048 knots one lane per
body, at most 1.25 times those of the three-role kernel, which works in body axes."""
import numpy as np
import pytest

from paper_2109_06976_amd import grid, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("more", [0, 1])
def test_end_of_the_range(orc, more):
    import torch
    n = 5
    robot = synth.random_model(synth.chain_parent(n), 60 + n, axes="random")
    N = 2 * torch.cuda.get_device_properties(0).multi_processor_count * (64 // n) + more
    m = grid.Model(robot)
    try:
        assert grid.kernel_for(m, N) == ("grid_fdgrad_serial_halves" if more
                                         else "grid_fdgrad_team_halves")
        print(f"[gpu] dFD, dID, VJP chain of {n} N={N}", flush=True)
        kn = synth.random_knots(n, N, 2600)
        g = synth.random_knots(n, N, 2601).qd
        q, qd, u, gb = (torch.from_numpy(a).cuda() for a in (kn.q, kn.qd, kn.tau, g))
        vec = [torch.full((N, n), float("nan"), device="cuda") for _ in range(4)]
        mat = [torch.full((N, n, n), float("nan"), device="cuda") for _ in range(5)]
        m.fd_grad(q, qd, u, vec[3], *mat[2:])
        m.id_grad(q, qd, u, *mat[:2])
        grid.fd_vjp_adjoint(m, q, qd, u, gb, *vec[:3])
        torch.cuda.synchronize()
        for t in vec + mat:
            assert bool(torch.isfinite(t).all())
        idx = np.unique(np.concatenate([[0, N - 1], np.random.default_rng(13).integers(0, N, 40)]))
        it = torch.from_numpy(idx).cuda()
        der = [orc.rnea_grad(robot, kn.q[k], kn.qd[k], kn.tau[k]) for k in idx]
        t = np.stack([orc.minv_cholesky(robot, kn.q[k]) @ g[k].astype(np.float64) for k in idx])
        fd = orc.fd_grad_batch(robot, kn.q[idx], kn.qd[idx], kn.tau[idx])
        want = [np.stack([-(a.T @ x) for (a, _), x in zip(der, t)]),
                np.stack([-(b.T @ x) for (_, b), x in zip(der, t)]), t, fd["qdd"],
                np.stack([a for a, _ in der]), np.stack([b for _, b in der]),
                fd["Minv"], fd["dqdd_dq"], fd["dqdd_dqd"]]
        for j, (ref, got) in enumerate(zip(want, vec + mat)):
            y = got[it].cpu().numpy().astype(np.float64)
            d, s = (np.abs(a).reshape(len(idx), -1).max(1) for a in (y - ref, ref))
            assert float((d / np.where(s > 0, s, 1.0)).max()) <= 1e-3, (n, N, j)
    finally:
        m.close()


def test_error_by_one_lane_per_body(orc):
    import torch
    n = 5
    robot = synth.random_model(synth.chain_parent(n), 60 + n, axes="random")
    kn = synth.random_knots(n, 2048, 2602)
    ins = [torch.from_numpy(a).cuda() for a in (kn.q, kn.qd, kn.tau)]
    ref = orc.fd_grad_batch(robot, kn.q, kn.qd, kn.tau)
    m = grid.Model(robot)
    err = {}
    try:
        for b in (grid.BUILD_PIPE, grid.BUILD_LANE_W2):
            print(f"[gpu] error of build {b}, chain of {n}", flush=True)
            grid.tune_apply(m, {1 << 22: b})
            out = grid.fd_grad_torch(m, *ins)
            torch.cuda.synchronize()
            err[b] = {k: float(np.linalg.norm(out[k].cpu().numpy().astype(np.float64) - ref[k]) /
                               np.linalg.norm(ref[k])) for k in out}
    finally:
        m.close()
    print({k: (err[grid.BUILD_PIPE][k], err[grid.BUILD_LANE_W2][k]) for k in ref}, flush=True)
    for k, e in err[grid.BUILD_LANE_W2].items():
        assert e <= 1.25 * err[grid.BUILD_PIPE][k], (n, k)
