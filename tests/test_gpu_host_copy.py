"""The host call on pinned buffers on both sides of the size where its copies change from a kernel
to the copy engines (8 MiB of outputs), and at one knot: bitwise the device call's outputs, the
phases timed."""
import numpy as np
import pytest

from paper_2109_06976_amd import grid, synth

pytestmark = pytest.mark.gpu

KEYS = ("qdd", "Minv", "dqdd_dq", "dqdd_dqd")


def test_pinned_call_around_the_copy_limit():
    import torch
    m = grid.Model(synth.chain7())
    n = m.n
    limit = (8 << 20) // (4 * (n + 3 * n * n))
    ws = grid.Workspace(m, limit + 1)
    try:
        for N in (1, limit, limit + 1):
            print(f"[gpu] pinned copies chain7 N={N}", flush=True)
            kn = synth.random_knots(n, N, 61)
            dev = grid.fd_grad_torch(m, *(torch.from_numpy(a).cuda() for a in (kn.q, kn.qd, kn.tau)))
            torch.cuda.synchronize()
            ins, outs = ws.host_buffers(N)
            ins["q"][:], ins["qd"][:], ins["tau"][:] = kn.q, kn.qd, kn.tau
            for o in outs.values():
                o.fill(np.nan)
            t = ws.fd_grad_pinned(N)
            assert min(t["h2d_ms"], t["kernel_ms"], t["d2h_ms"]) > 0
            for k in KEYS:
                np.testing.assert_array_equal(outs[k], dev[k].cpu().numpy())
    finally:
        ws.close()
        m.close()
