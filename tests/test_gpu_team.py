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
