"""The kernels with one lane per body against the FP64 oracle on an MI355X, at knot counts
around the number of knots a wavefront holds (64 / (branches of a shape x their bodies): one
knot less, as many, one more, and two wavefronts and one knot), into output arrays filled with
NaN at an address one float past a 16-byte boundary. The tolerances are those of the parity
tests (normwise per knot: vectors 1e-4, matrices 1e-3).
"""
import sys

import numpy as np
import pytest

from paper_2109_06976_amd import grid, synth
from paper_2109_06976_amd.build import max_size_model, prismatic_models, star_model

pytestmark = pytest.mark.gpu

TOL = {"qdd": 1e-4, "Minv": 1e-3, "dqdd_dq": 1e-3, "dqdd_dqd": 1e-3}

# robot, knots per wavefront of its largest shape
ROBOTS = {
    "chain1": (lambda: synth.random_model(synth.chain_parent(1), 40), 64),
    "chain7": (synth.chain7, 9),
    "quad12": (synth.quad12, 5),              # four branches of one shape side by side
    "humanoid30": (synth.humanoid30, 3),      # an 18-body branch; two of 6 side by side
    "humanoid32": (max_size_model, 3),        # a 20-body branch
    "tree5-axes-prism": (lambda: prismatic_models()["tree5-axes-prism"], 16),
    "star32": (star_model, 2),                # 32 branches of one body
}


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def shifted(torch, *shape):
    """A NaN-filled array one float past an aligned address, with guards on both sides."""
    size = int(np.prod(shape))
    base = torch.full((size + 8,), float("nan"), device="cuda")
    return base, base[1:1 + size].view(shape), size


def check(name, got, ref, tol):
    N = ref.shape[0]
    d = np.abs(got.astype(np.float64) - ref).reshape(N, -1).max(1)
    s = np.abs(ref).reshape(N, -1).max(1)
    err = float((d / np.where(s > 0, s, 1.0)).max())
    assert err <= tol, (name, err)


@pytest.mark.parametrize("name", list(ROBOTS))
def test_team_gradient_at_wavefront_edges(orc, name):
    import torch
    make, K = ROBOTS[name]
    robot = make()
    n = robot.n
    m = grid.Model(robot)
    try:
        grid.tune_apply(m, {1 << 22: grid.BUILD_LANE})
        for N in sorted({max(1, K - 1), K, K + 1, 2 * K + 1}):
            say(f"[gpu] team gradient {name} N={N}")
            kn = synth.random_knots(n, N, 1400 + N)
            ins = [torch.from_numpy(a).cuda() for a in (kn.q, kn.qd, kn.tau)]
            bufs = [shifted(torch, N, n)] + [shifted(torch, N, n, n) for _ in range(3)]
            m.fd_grad(*ins, *(b[1] for b in bufs), N=N)
            torch.cuda.synchronize()
            ref = orc.fd_grad_batch(robot, kn.q, kn.qd, kn.tau)
            for (key, tol), (base, out, size) in zip(TOL.items(), bufs):
                check((name, N, key), out.cpu().numpy(), ref[key], tol)
                assert bool(torch.isnan(base[:1]).all()) and bool(torch.isnan(base[1 + size:]).all())
            Mi = bufs[1][1].cpu().numpy()
            np.testing.assert_array_equal(Mi, np.swapaxes(Mi, 1, 2))
    finally:
        m.close()


@pytest.mark.parametrize("name", list(ROBOTS))
def test_team_algorithms_on_large_batches(orc, name):
    """FD, M^-1, dID and the adjoint VJP at a batch that takes them to one lane per body on any
    robot (more than two wavefronts per SIMD of the quad layout: 64 sampled knots, the first and
    the last included, against the oracle), the other knots finite."""
    import torch
    make, _ = ROBOTS[name]
    robot = make()
    n = robot.n
    N = 256 * torch.cuda.get_device_properties(0).multi_processor_count + 3
    m = grid.Model(robot)
    try:
        say(f"[gpu] team algorithms {name} N={N}")
        kn = synth.random_knots(n, N, 1500)
        g = synth.random_knots(n, N, 1501).qd
        q, qd, tau, gb = (torch.from_numpy(a).cuda() for a in (kn.q, kn.qd, kn.tau, g))
        vec = [torch.full((N, n), float("nan"), device="cuda") for _ in range(4)]
        mat = [torch.full((N, n, n), float("nan"), device="cuda") for _ in range(3)]
        m.fd(q, qd, tau, vec[0])
        m.minv(q, mat[0])
        m.id_grad(q, qd, tau, mat[1], mat[2])
        grid.fd_vjp_adjoint(m, q, qd, tau, gb, vec[1], vec[2], vec[3])
        torch.cuda.synchronize()
        for t in vec + mat:
            assert bool(torch.isfinite(t).all())
        idx = np.unique(np.concatenate([[0, N - 1], np.random.default_rng(7).integers(0, N, 62)]))
        it = torch.from_numpy(idx).cuda()
        fd, qb, qdb, tb = (t[it].cpu().numpy() for t in vec)
        mi, dq, dqd = (t[it].cpu().numpy() for t in mat)
        r_fd, r_mi, r_dq, r_dqd, r_v = [], [], [], [], []
        for k in idx:
            r_fd.append(orc.fd(robot, kn.q[k], kn.qd[k], kn.tau[k]))
            r_mi.append(orc.minv_cholesky(robot, kn.q[k]))
            a, b = orc.rnea_grad(robot, kn.q[k], kn.qd[k], kn.tau[k])
            r_dq.append(a)
            r_dqd.append(b)
            t = r_mi[-1] @ g[k].astype(np.float64)
            r_v.append((-(a.T @ t), -(b.T @ t), t))
        check((name, "FD"), fd, np.stack(r_fd), 1e-4)
        check((name, "Minv"), mi, np.stack(r_mi), 1e-3)
        check((name, "dID dq"), dq, np.stack(r_dq), 1e-3)
        check((name, "dID dqd"), dqd, np.stack(r_dqd), 1e-3)
        for got, ref, what in zip((qb, qdb, tb), zip(*r_v), ("qbar", "qdbar", "taubar")):
            check((name, what), got, np.stack(ref), 1e-3)
        np.testing.assert_array_equal(mi, np.swapaxes(mi, 1, 2))
    finally:
        m.close()
