"""Every native launch against the ctypes call of the same library function on an MI355X, on a stream
of its own: outputs and gradients bit for bit. The ctypes side is forced by denying that tensors are
plain, which is what the wrappers ask before they take the native path."""
import pytest

from paper_2109_06976_amd import grid, synth

pytestmark = pytest.mark.gpu

N, n = 37, 7


@pytest.fixture(scope="module")
def model():
    import torch  # noqa: F401
    m = grid.Model(synth.chain7())
    yield m
    m.close()


def both(monkeypatch, call):
    """call() by the native launches, then by ctypes, each on the same side stream"""
    import torch
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    runs, native = [], []
    real = grid._native()
    for plain in (True, False):
        with monkeypatch.context() as mp, torch.cuda.stream(side):
            if not plain:
                mp.setattr(grid, "_plain_torch", lambda x: False)
            runs.append(call(side))
        torch.cuda.synchronize()
        native.append(plain)
    assert real is grid._native()
    for a, b in zip(*runs):
        assert bool(torch.isfinite(a).all()) and torch.equal(a, b)


def data(torch, requires_grad=False):
    kn = synth.random_knots(n, N, 6)
    x = [torch.from_numpy(a).cuda() for a in (kn.q, kn.qd, kn.tau)]
    return [t.requires_grad_(requires_grad) for t in x]


def empty(torch, *shape):
    return torch.full(shape, float("nan"), device="cuda")


LAUNCHES = {
    "fd_grad": lambda m, t, x, s: (lambda o: (m.fd_grad(*x, *o, stream=s), o)[1])(
        [empty(t, N, n)] + [empty(t, N, n, n) for _ in range(3)]),
    "id": lambda m, t, x, s: (lambda o: (m.id(*x, o, stream=s), [o])[1])(empty(t, N, n)),
    "fd": lambda m, t, x, s: (lambda o: (m.fd(*x, o, stream=s), [o])[1])(empty(t, N, n)),
    "minv": lambda m, t, x, s: (lambda o: (m.minv(x[0], o, stream=s), [o])[1])(empty(t, N, n, n)),
    "id_grad": lambda m, t, x, s: (lambda o: (m.id_grad(*x, *o, stream=s), o)[1])(
        [empty(t, N, n, n) for _ in range(2)]),
    "fd_vjp_adjoint": lambda m, t, x, s: (lambda o: (
        grid.fd_vjp_adjoint(m, *x, x[1], *o, stream=s), o)[1])([empty(t, N, n) for _ in range(3)]),
    "fd_vjp": lambda m, t, x, s: (lambda d, o: (
        grid.fd_vjp(m, d["dqdd_dq"], d["dqdd_dqd"], d["Minv"], x[1], *o, stream=s), o)[1])(
        grid.fd_grad_torch(m, *x), [empty(t, N, n) for _ in range(3)]),
    "fd_grad_torch": lambda m, t, x, s: list(grid.fd_grad_torch(m, *x).values()),
}


@pytest.mark.parametrize("name", list(LAUNCHES))
def test_launch_equals_ctypes(model, monkeypatch, name):
    import torch
    x = data(torch)
    print(f"[gpu] native and ctypes {name}", flush=True)
    both(monkeypatch, lambda s: LAUNCHES[name](model, torch, x, s))


@pytest.mark.parametrize("mode", ["jacobians", "adjoint"])
def test_backward_equals_ctypes(model, monkeypatch, mode):
    import torch
    from paper_2109_06976_amd import autograd
    x = data(torch, requires_grad=True)
    g = torch.linspace(-1.0, 1.0, N * n, device="cuda").view(N, n)

    def step(_):
        qdd = autograd.forward_dynamics(model, *x, mode)
        return [qdd.detach(), *torch.autograd.grad(qdd, x, g)]

    print(f"[gpu] native and ctypes step, {mode}", flush=True)
    both(monkeypatch, step)
