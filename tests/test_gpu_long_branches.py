"""Branches of 9 to 17 bodies on an MI355X: the gradient keeps the three-role kernel while the
wavefronts of such branches fit one per SIMD, and FD, M^-1, dID and the adjoint VJP keep the quad
layout for small batches. Each algorithm on both sides of its line, and with one lane per body on
trees whose rows lie among other branches', against the FP64 oracle at sampled knots, the first and
the last included; outputs start as NaN. The tolerances are those of the parity tests (normwise per
knot: vectors 1e-4, matrices 1e-3)."""
import numpy as np
import pytest

from paper_2109_06976_amd import grid, synth
from paper_2109_06976_amd.build import tree_models

pytestmark = pytest.mark.gpu


def check(name, got, ref, tol):
    N = ref.shape[0]
    d = np.abs(got.astype(np.float64) - ref).reshape(N, -1).max(1)
    s = np.abs(ref).reshape(N, -1).max(1)
    err = float((d / np.where(s > 0, s, 1.0)).max())
    assert err <= tol, (name, err)


def sample(N, seed):
    return np.unique(np.concatenate([[0, N - 1], np.random.default_rng(seed).integers(0, N, 30)]))


@pytest.mark.parametrize("name", ["branches13", "chain17"])
def test_gradient_on_both_sides_of_the_three_role_kernels_line(orc, name):
    import torch
    robot = tree_models()[name]
    m = grid.Model(robot)
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    try:
        # four wavefronts per knot of the one long branch: as many knots as compute units
        assert [grid.kernel_for(m, N) for N in (1, 9, cu, cu + 1)] == \
            ["grid_fdgrad_pipe"] * 3 + ["grid_fdgrad_team_halves"]
        for N in (9, cu, cu + 1):
            print(f"[gpu] dFD {name} N={N}", flush=True)
            kn = synth.random_knots(robot.n, N, 2200 + N)
            out = grid.fd_grad_torch(m, *(torch.from_numpy(a).cuda() for a in (kn.q, kn.qd, kn.tau)))
            torch.cuda.synchronize()
            ref = orc.fd_grad_batch(robot, kn.q, kn.qd, kn.tau)
            for k in out:
                check((name, N, k), out[k].cpu().numpy(), ref[k], 1e-4 if k == "qdd" else 1e-3)
    finally:
        m.close()


def test_shallow_long_branch_runs_one_lane_per_body_beyond_a_few_knots():
    import torch  # noqa: F401
    m = grid.Model(synth.humanoid30())
    try:
        assert {grid.kernel_for(m, N) for N in (1, 8)} == {"grid_fdgrad_pipe"}
        assert {grid.kernel_for(m, N) for N in (9, 128)} == {"grid_fdgrad_team_halves"}
    finally:
        m.close()


# knots per compute unit: below and beyond each line (FD 4, M^-1 8, dID 1, VJP 4 of branches13; FD
# and M^-1 none, dID 1, VJP 4 of chain17), and one lane per body or problem on pairs8
@pytest.mark.parametrize("per_cu", [0.1, 1, 4, 8.5])
@pytest.mark.parametrize("name", ["branches13", "chain17", "pairs8"])
def test_algorithms_around_their_lines(orc, name, per_cu):
    import torch
    robot = tree_models()[name]
    n = robot.n
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    m = grid.Model(robot)
    try:
        for N in (int(per_cu * cu), int(per_cu * cu) + 1):
            print(f"[gpu] FD, M^-1, dID, VJP {name} N={N}", flush=True)
            kn = synth.random_knots(n, N, 2300)
            g = synth.random_knots(n, N, 2301).qd
            q, qd, tau, gb = (torch.from_numpy(a).cuda() for a in (kn.q, kn.qd, kn.tau, g))
            vec = [torch.full((N, n), float("nan"), device="cuda") for _ in range(4)]
            mat = [torch.full((N, n, n), float("nan"), device="cuda") for _ in range(3)]
            m.fd(q, qd, tau, vec[0])
            m.minv(q, mat[0])
            m.id_grad(q, qd, tau, mat[1], mat[2])
            grid.fd_vjp_adjoint(m, q, qd, tau, gb, *vec[1:])
            torch.cuda.synchronize()
            for t in vec + mat:
                assert bool(torch.isfinite(t).all())
            idx = sample(N, 11)
            it = torch.from_numpy(idx).cuda()
            fd, qb, qdb, tb = (t[it].cpu().numpy() for t in vec)
            mi, dq, dqd = (t[it].cpu().numpy() for t in mat)
            r_mi = np.stack([orc.minv_cholesky(robot, kn.q[k]) for k in idx])
            der = [orc.rnea_grad(robot, kn.q[k], kn.qd[k], kn.tau[k]) for k in idx]
            r_t = (r_mi @ g[idx].astype(np.float64)[..., None])[..., 0]
            check((name, N, "FD"), fd,
                  np.stack([orc.fd(robot, kn.q[k], kn.qd[k], kn.tau[k]) for k in idx]), 1e-4)
            check((name, N, "Minv"), mi, r_mi, 1e-3)
            check((name, N, "dID dq"), dq, np.stack([a for a, _ in der]), 1e-3)
            check((name, N, "dID dqd"), dqd, np.stack([b for _, b in der]), 1e-3)
            check((name, N, "taubar"), tb, r_t, 1e-3)
            check((name, N, "qbar"), qb, np.stack([-(a.T @ t) for (a, _), t in zip(der, r_t)]), 1e-3)
            check((name, N, "qdbar"), qdb, np.stack([-(b.T @ t) for (_, b), t in zip(der, r_t)]), 1e-3)
            np.testing.assert_array_equal(mi, np.swapaxes(mi, 1, 2))
    finally:
        m.close()
