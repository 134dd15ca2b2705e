"""The native forward-dynamics node under saved-tensor hooks on an MI355X: what the caller's unpack
hook returns is checked like an argument before a launch, and a region under checkpointing is
recomputed in the unpack hook with its graph."""
import pytest

from paper_2109_06976_amd import grid, synth

pytestmark = pytest.mark.gpu

N = 37


@pytest.fixture(scope="module")
def model():
    import torch  # noqa: F401  (before the library: both then share one HIP runtime)
    m = grid.Model(synth.chain7())
    yield m
    m.close()


def inputs(torch, seed=5):
    kn = synth.random_knots(7, N, seed)
    return [torch.from_numpy(a).cuda().requires_grad_(True) for a in (kn.q, kn.qd, kn.tau)]


def strided(t):
    """The same values, every other element of a wider array."""
    wide = t.new_empty((*t.shape, 2))
    wide[..., 0] = t
    return wide[..., 0]


UNPACK = {"half": lambda t: t.half(), "short": lambda t: t[:-1].contiguous(), "strided": strided,
          "host": lambda t: t.cpu()}


@pytest.mark.parametrize("kind", list(UNPACK))
@pytest.mark.parametrize("mode", ["jacobians", "adjoint"])
def test_backward_refuses_unpacked_tensors_that_do_not_fit(model, mode, kind):
    import torch
    from paper_2109_06976_amd import autograd
    ins = inputs(torch)
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t, UNPACK[kind]):
        qdd = autograd.forward_dynamics(model, *ins, mode)
    print(f"[gpu] unpacked {kind}, {mode}", flush=True)
    with pytest.raises(grid.GridError) as e:
        torch.autograd.grad(qdd, ins, torch.ones_like(qdd))
    assert e.value.status == grid.GRID_EINVAL


@pytest.mark.parametrize("mode", ["jacobians", "adjoint"])
def test_checkpointed_region_is_recomputed_with_its_graph(model, mode):
    import torch
    from torch.utils.checkpoint import checkpoint
    from paper_2109_06976_amd import autograd
    ins = inputs(torch)

    def region(q, qd, tau):
        # what precedes the node saves tensors of its own; the Euler step after it saves none
        qdd = autograd.forward_dynamics(model, q.sin() * q, qd, tau, mode)
        return qd + 0.01 * qdd

    w = torch.linspace(-1.0, 1.0, 7, device="cuda")
    print(f"[gpu] checkpointed region, {mode}", flush=True)
    want = torch.autograd.grad((region(*ins) * w).sum(), ins)
    got = torch.autograd.grad((checkpoint(region, *ins, use_reentrant=False) * w).sum(), ins)
    for a, b in zip(got, want):
        assert torch.equal(a, b)


@pytest.mark.parametrize("mode", ["jacobians", "adjoint"])
def test_backward_raises_the_library_error(mode):
    import torch
    from paper_2109_06976_amd import autograd
    m = grid.Model(synth.chain7())
    ins = inputs(torch)
    qdd = autograd.forward_dynamics(m, *ins, mode)
    torch.cuda.synchronize()
    m.close()
    print(f"[gpu] model closed before the backward step, {mode}", flush=True)
    with pytest.raises(grid.GridError) as e:
        torch.autograd.grad(qdd, ins, torch.ones_like(qdd))
    assert e.value.status == grid.GRID_EINVAL
