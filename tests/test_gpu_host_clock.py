"""The host call timed by the copy kernels' clock values: batches whose copies end in 0 to 3 floats
beyond the 16-byte pieces and take one, two and many workgroups, with and without timing bitwise
the device call's outputs; the phases are positive, add up to the total and lie within the call."""
import ctypes as C
import time

import numpy as np
import pytest

from paper_2109_06976_amd import grid, synth

pytestmark = pytest.mark.gpu

KEYS = ("qdd", "Minv", "dqdd_dq", "dqdd_dqd")


def test_host_call_with_and_without_timing():
    import torch
    m = grid.Model(synth.chain7())
    n = m.n
    ws = grid.Workspace(m, 1200)
    try:
        for N in (1, 2, 3, 4, 6, 7, 13, 300, 1200):
            print(f"[gpu] host call chain7 N={N}", flush=True)
            kn = synth.random_knots(n, N, 62)
            dev = grid.fd_grad_torch(m, *(torch.from_numpy(a).cuda() for a in (kn.q, kn.qd, kn.tau)))
            torch.cuda.synchronize()
            begin = time.perf_counter()
            host, t = ws.fd_grad_host(kn.q, kn.qd, kn.tau)
            wall = 1e3 * (time.perf_counter() - begin)
            for k in KEYS:
                np.testing.assert_array_equal(host[k], dev[k].cpu().numpy())
            phases = [t["h2d_ms"], t["kernel_ms"], t["d2h_ms"]]
            assert min(phases) > 0 and t["total_ms"] <= wall
            assert abs(sum(phases) - t["total_ms"]) <= 1e-5 * t["total_ms"] + 1e-6
            ins, outs = ws.host_buffers(N)
            ins["q"][:], ins["qd"][:], ins["tau"][:] = kn.q, kn.qd, kn.tau
            for o in outs.values():
                o.fill(np.nan)
            status = grid.lib().grid_fd_grad_pinned(m.handle, ws._h, N, 1, C.POINTER(grid.GridTiming)())
            assert status == grid.GRID_OK
            for k in KEYS:
                np.testing.assert_array_equal(outs[k], dev[k].cpu().numpy())
    finally:
        ws.close()
        m.close()
