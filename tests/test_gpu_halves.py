"""One lane per problem with half of the outputs on each of two wavefronts (dFD as build 5, dID),
and ID in that layout, against the FP64 oracle on an MI355X, at knot counts around the 64 of a
wavefront and at batches that choose these kernels, the first and the last knot included; outputs
start as NaN. The tolerances are those of the parity tests (normwise per knot: vectors 1e-4,
matrices 1e-3).
"""
import numpy as np
import pytest

from paper_2109_06976_amd import grid, synth
from paper_2109_06976_amd.build import prismatic_models

pytestmark = pytest.mark.gpu

ROBOTS = {
    "chain7": synth.chain7,
    "quad12": synth.quad12,                   # four branches, rows of each among the others'
    "chain1": lambda: synth.random_model(synth.chain_parent(1), 40),
    "tree5-axes-prism": lambda: prismatic_models()["tree5-axes-prism"],
}


def check(name, got, ref, tol):
    N = ref.shape[0]
    d = np.abs(got.astype(np.float64) - ref).reshape(N, -1).max(1)
    s = np.abs(ref).reshape(N, -1).max(1)
    err = float((d / np.where(s > 0, s, 1.0)).max())
    assert err <= tol, (name, err)


@pytest.mark.parametrize("build", [grid.BUILD_SERIAL, grid.BUILD_SERIAL2])
@pytest.mark.parametrize("name", list(ROBOTS))
def test_gradient_in_halves_and_whole(orc, name, build):
    import torch
    robot = ROBOTS[name]()
    n = robot.n
    m = grid.Model(robot)
    try:
        grid.tune_apply(m, {1 << 22: build})
        for N in (1, 63, 64, 65, 131):
            print(f"[gpu] dFD build {build} {name} N={N}", flush=True)
            kn = synth.random_knots(n, N, 1700 + N)
            ins = [torch.from_numpy(a).cuda() for a in (kn.q, kn.qd, kn.tau)]
            outs = [torch.full((N, n) + (n,) * (k > 0), float("nan"), device="cuda")
                    for k in range(4)]
            m.fd_grad(*ins, *outs, N=N)
            torch.cuda.synchronize()
            ref = orc.fd_grad_batch(robot, kn.q, kn.qd, kn.tau)
            for key, out in zip(("qdd", "Minv", "dqdd_dq", "dqdd_dqd"), outs):
                check((name, N, key), out.cpu().numpy(), ref[key], 1e-4 if key == "qdd" else 1e-3)
    finally:
        m.close()


@pytest.mark.parametrize("per_cu", [60, 257])
@pytest.mark.parametrize("name", list(ROBOTS))
def test_inverse_dynamics_on_large_batches(orc, name, per_cu):
    import torch
    robot = ROBOTS[name]()
    n = robot.n
    N = per_cu * torch.cuda.get_device_properties(0).multi_processor_count + 3
    m = grid.Model(robot)
    try:
        print(f"[gpu] ID, dID {name} N={N}", flush=True)
        kn = synth.random_knots(n, N, 1800)
        q, qd, qdd = (torch.from_numpy(a).cuda() for a in (kn.q, kn.qd, kn.tau))
        tau = torch.full((N, n), float("nan"), device="cuda")
        dq, dqd = (torch.full((N, n, n), float("nan"), device="cuda") for _ in range(2))
        m.id(q, qd, qdd, tau)
        m.id_grad(q, qd, qdd, dq, dqd)
        torch.cuda.synchronize()
        for t in (tau, dq, dqd):
            assert bool(torch.isfinite(t).all())
        idx = np.unique(np.concatenate([[0, N - 1], np.random.default_rng(8).integers(0, N, 62)]))
        it = torch.from_numpy(idx).cuda()
        ref = [orc.rnea_grad(robot, kn.q[k], kn.qd[k], kn.tau[k]) for k in idx]
        check((name, "ID"), tau[it].cpu().numpy(),
              np.stack([orc.rnea(robot, kn.q[k], kn.qd[k], kn.tau[k]) for k in idx]), 1e-4)
        check((name, "dID dq"), dq[it].cpu().numpy(), np.stack([a for a, _ in ref]), 1e-3)
        check((name, "dID dqd"), dqd[it].cpu().numpy(), np.stack([b for _, b in ref]), 1e-3)
    finally:
        m.close()


@pytest.mark.parametrize("build", [grid.BUILD_LANE, grid.BUILD_LANE_W2])
@pytest.mark.parametrize("name", ["chain7", "humanoid30", "humanoid30-prism"])
def test_gradient_by_bodies_in_halves_and_whole(orc, name, build):
    import torch
    robot = {**prismatic_models(), "chain7": synth.chain7(), "humanoid30": synth.humanoid30()}[name]
    n = robot.n
    m = grid.Model(robot)
    try:
        grid.tune_apply(m, {1 << 22: build})
        for N in (1, 9, 10, 61):
            print(f"[gpu] dFD build {build} {name} N={N}", flush=True)
            kn = synth.random_knots(n, N, 1900 + N)
            ins = [torch.from_numpy(a).cuda() for a in (kn.q, kn.qd, kn.tau)]
            outs = [torch.full((N, n) + (n,) * (k > 0), float("nan"), device="cuda")
                    for k in range(4)]
            m.fd_grad(*ins, *outs, N=N)
            torch.cuda.synchronize()
            ref = orc.fd_grad_batch(robot, kn.q, kn.qd, kn.tau)
            for key, out in zip(("qdd", "Minv", "dqdd_dq", "dqdd_dqd"), outs):
                check((name, N, key), out.cpu().numpy(), ref[key], 1e-4 if key == "qdd" else 1e-3)
    finally:
        m.close()
