"""The native torch-facing calls against the Python path on an MI355X: the same outputs and
gradients bit for bit, saved-tensor hooks seen, and the same refusals. What is not a plain
contiguous float32 tensor on the model's device goes the Python way.
"""
import numpy as np
import pytest

from paper_2109_06976_amd import grid, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def setup():
    import torch
    model = grid.Model(synth.chain7())
    kn = synth.random_knots(7, 37, 5)
    yield model, [torch.from_numpy(a).cuda() for a in (kn.q, kn.qd, kn.tau)]
    model.close()


@pytest.mark.parametrize("mode", ["jacobians", "adjoint"])
def test_native_step_equals_python_step(setup, mode):
    import torch
    from paper_2109_06976_amd import autograd
    model, x = setup
    g = torch.randn_like(x[0])
    runs, seen = [], []

    def pack(t):
        seen.append(t.shape)
        return t

    for call in (lambda *a: autograd.forward_dynamics(model, *a, mode),
                 lambda *a: autograd.ForwardDynamics.apply(*a, model, mode)):
        ins = [t.clone().requires_grad_(True) for t in x]
        with torch.autograd.graph.saved_tensors_hooks(pack, lambda t: t):
            qdd = call(*ins)
        runs.append([qdd.detach(), *torch.autograd.grad(qdd, ins, g)])
    assert len(seen) == 6 and seen[:3] == seen[3:]
    for a, b in zip(*runs):
        assert torch.equal(a, b)
    # only some of the inputs differentiable; none
    ins = [x[0], x[1].clone().requires_grad_(True), x[2]]
    (got,) = torch.autograd.grad(autograd.forward_dynamics(model, *ins, mode), ins[1:2], g)
    assert torch.equal(got, runs[0][2])
    assert not autograd.forward_dynamics(model, *x, mode).requires_grad


def test_native_gradient_equals_python_path(setup):
    import torch
    model, x = setup
    a = grid.fd_grad_torch(model, *x)
    # strided and float64 inputs are converted by the Python path
    wide = [torch.stack((t, t), -1)[..., 0] for t in x]
    b = grid.fd_grad_torch(model, *wide)
    c = grid.fd_grad_torch(model, *(t.double() for t in x))
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        d = grid.fd_grad_torch(model, *x)
    e = grid.fd_grad_torch(model, *x, stream=side)
    torch.cuda.synchronize()
    for k in a:
        for o in (b, c, d, e):
            assert o[k].dtype == torch.float32 and torch.equal(a[k], o[k])
    empty = grid.fd_grad_torch(model, *(t[:0] for t in x))
    assert empty["Minv"].shape == (0, 7, 7)


def test_native_calls_refuse_what_the_python_path_refuses(setup):
    import torch
    from paper_2109_06976_amd import autograd
    model, x = setup
    short = torch.empty((36, 7), device="cuda")
    with pytest.raises(ValueError):               # torch: no stream of a host device
        grid.fd_grad_torch(model, *(t.cpu() for t in x))
    for call in (lambda: grid.fd_grad_torch(model, x[0], x[1], short),
                 lambda: model.id(*x, short),
                 lambda: model.minv(x[0], torch.empty((37, 7, 7))),
                 lambda: model.fd(x[0], x[1], x[2].double(), torch.empty_like(x[0])),
                 lambda: model.id(*x, torch.empty_like(x[0]), N=-1),
                 lambda: autograd.forward_dynamics(model, x[0], x[1], short)):
        with pytest.raises(grid.GridError) as e:
            call()
        assert e.value.status == grid.GRID_EINVAL
    with pytest.raises(ValueError):
        autograd.forward_dynamics(model, *x, "other")
    # a model closed between forward and backward: an error, no use of its handle
    m = grid.Model(synth.chain7())
    ins = [t.clone().requires_grad_(True) for t in x]
    qdd = autograd.forward_dynamics(m, *ins)
    torch.cuda.synchronize()
    m.close()
    with pytest.raises(RuntimeError, match="GRID_EINVAL"):
        torch.autograd.grad(qdd, ins, torch.ones_like(qdd))
    with pytest.raises(grid.GridError):
        grid.fd_grad_torch(m, *x)
    # transforms see the Python function, which has no rule for them, as before
    with pytest.raises(RuntimeError):
        torch.func.vmap(lambda a: autograd.forward_dynamics(model, a[None], a[None], a[None]))(x[0])
    assert np.isfinite(x[0].cpu().numpy()).all()
