"""Branches of one and two bodies on an MI355X: an untuned model goes from the three-role kernel to one
lane per problem, without the quad kernel, which is slower there; both kernels give the same gradient
of the same knots (each batch half of the other's)."""
import pytest

from paper_2109_06976_amd import grid, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, N", [(1, 8192), (2, 4096)])
def test_short_chains_beyond_the_three_role_kernel(n, N):
    import torch
    m = grid.Model(synth.random_model(synth.chain_parent(n), 39 + n))
    try:
        N = N * torch.cuda.get_device_properties(0).multi_processor_count // 256
        assert grid.kernel_for(m, N // 2) == "grid_fdgrad_pipe"
        assert grid.kernel_for(m, N) == "grid_fdgrad_serial_halves"
        print(f"[gpu] dFD chain of {n}, N={N}", flush=True)
        kn = synth.random_knots(n, N, 2400)
        ins = [torch.from_numpy(a).cuda() for a in (kn.q, kn.qd, kn.tau)]
        whole = grid.fd_grad_torch(m, *ins)
        parts = [grid.fd_grad_torch(m, *(t[k:k + N // 2].contiguous() for t in ins))
                 for k in (0, N // 2)]
        for k, y in whole.items():
            ref = torch.cat([p[k] for p in parts])
            # float32 roundings of up to some hundred operations, by the norm of the batch
            assert float((y - ref).norm()) <= 1e-5 * float(ref.norm()), k
    finally:
        m.close()
