"""The discrete-time Jacobians on an MI355X: dt dqdd/dq and dt M^-1 enter A and B as one product each,
bit for bit, the sign of a zero included."""
import pytest

from paper_2109_06976_amd import grid, synth

pytestmark = pytest.mark.gpu


def test_products_keep_the_sign_of_zero():
    import torch
    m = grid.Model(synth.chain7())
    n, N, dt = 7, 37, 0.01
    try:
        print("[gpu] discrete-time Jacobians with signed zeros", flush=True)
        g = torch.Generator(device="cuda")
        g.manual_seed(3)
        dq, dqd, mi = (torch.randn((N, n, n), generator=g, device="cuda") for _ in range(3))
        for t in (dq, dqd, mi):
            t[::2, 0] = -0.0
            t[::3, 1] = 0.0
        A, B = torch.empty((N, 2 * n, 2 * n), device="cuda"), torch.empty((N, 2 * n, n), device="cuda")
        grid.dt_jacobians(m, dt, dq, dqd, mi, A, B)
        torch.cuda.synchronize()
        h = torch.tensor(dt, device="cuda")              # float32, as the kernel's
        bits = lambda x: x.contiguous().view(torch.int32)
        assert torch.equal(bits(A[:, n:, :n]), bits(h * dq))
        assert torch.equal(bits(B[:, n:]), bits(h * mi))
        assert torch.equal(bits(B[:, :n]), bits(h * h * mi))
    finally:
        m.close()
