"""grid_dt_jacobians on an MI355X against the formula in float64 on random matrices, at one to 32
joints and knot counts around the number that a workgroup takes (1024 / n^2, at least 1).

Each entry is one product with a rounded factor (dt or dt^2) and at most one sum: its error is at
most two roundings of the product and one of the result, 4 x 2^-24 of the sum of magnitudes.
"""
import numpy as np
import pytest

from paper_2109_06976_amd import grid, synth
from paper_2109_06976_amd.build import max_size_model

pytestmark = pytest.mark.gpu

ROBOTS = {"chain1": lambda: synth.random_model(synth.chain_parent(1), 40),
          "chain7": synth.chain7, "quad12": synth.quad12, "humanoid32": max_size_model}


@pytest.mark.parametrize("name", list(ROBOTS))
def test_dt_jacobians_at_workgroup_edges(name):
    import torch
    m = grid.Model(ROBOTS[name]())
    n = m.n
    K = max(1, 1024 // (n * n))
    dt = np.float64(np.float32(0.01))
    try:
        for N in sorted({1, max(1, K - 1), K, K + 1, 3 * K + 2}):
            print(f"[gpu] dt jacobians {name} N={N}", flush=True)
            rng = np.random.default_rng(N)
            Dq, Dqd, Mi = (rng.standard_normal((N, n, n)).astype(np.float32) * 50 for _ in range(3))
            A = torch.full((N, 2 * n, 2 * n), float("nan"), device="cuda")
            B = torch.full((N, 2 * n, n), float("nan"), device="cuda")
            grid.dt_jacobians(m, 0.01, *(torch.from_numpy(x).cuda() for x in (Dq, Dqd, Mi)), A, B)
            torch.cuda.synchronize()
            eye = np.broadcast_to(np.eye(n), (N, n, n))
            z = np.zeros((N, n, n))
            parts = [[(eye, dt * dt * Dq), (dt * eye, dt * dt * Dqd)], [(z, dt * Dq), (eye, dt * Dqd)]]
            for r in range(2):
                for c in range(2):
                    a, b = parts[r][c]
                    got = A[:, r * n:(r + 1) * n, c * n:(c + 1) * n].cpu().numpy().astype(np.float64)
                    assert np.all(np.abs(got - (a + b)) <= 4 * 2.0 ** -24 * (np.abs(a) + np.abs(b)))
            for r, f in enumerate((dt * dt, dt)):
                got = B[:, r * n:(r + 1) * n].cpu().numpy().astype(np.float64)
                assert np.all(np.abs(got - f * Mi) <= 4 * 2.0 ** -24 * np.abs(f * Mi))
    finally:
        m.close()
