"""A knot with NaN or infinite inputs leaves the knots beside it alone on an MI355X: where a wavefront
holds several knots, their outputs are bit for bit those of a batch without that knot's values."""
import pytest

from paper_2109_06976_amd import grid, synth
from paper_2109_06976_amd.build import tree_models

pytestmark = pytest.mark.gpu

N, BAD = 37, 4
VALUES = {"nan": float("nan"), "inf": float("inf")}
ROBOTS = {"chain7": synth.chain7, "quad12": synth.quad12, "humanoid30": synth.humanoid30,
          "pairs8": lambda: tree_models()["pairs8"], "branches13": lambda: tree_models()["branches13"]}


@pytest.mark.parametrize("value", list(VALUES))
@pytest.mark.parametrize("which", ["q", "qd", "tau"])
@pytest.mark.parametrize("name", list(ROBOTS))
def test_other_knots_are_untouched(name, which, value):
    import torch
    m = grid.Model(ROBOTS[name]())
    n = m.n
    others = torch.arange(N, device="cuda") != BAD
    try:
        kn = synth.random_knots(n, N, 2600)
        clean = [torch.from_numpy(a).cuda() for a in (kn.q, kn.qd, kn.tau)]
        dirty = [t.clone() for t in clean]
        dirty[("q", "qd", "tau").index(which)][BAD, ::2] = VALUES[value]

        def algorithms(x):
            v = [torch.empty((N, n), device="cuda") for _ in range(5)]
            a = [torch.empty((N, n, n), device="cuda") for _ in range(3)]
            m.id(*x, v[0])
            m.fd(*x, v[1])
            m.minv(x[0], a[0])
            m.id_grad(*x, a[1], a[2])
            grid.fd_vjp_adjoint(m, *x, clean[1], *v[2:])
            return v + a

        def gradient(x):
            return list(grid.fd_grad_torch(m, *x).values())

        calls = [("algorithms", -1, algorithms)]
        calls += [("gradient", b, gradient) for b in (0, 1, 2, 4, 5, 7)]
        for what, build, call in calls:
            grid.tune_apply(m, {1 << 22: build} if build >= 0 else {})
            print(f"[gpu] {name} {which}={value}: {what}, build {build}", flush=True)
            a, b = call(clean), call(dirty)
            torch.cuda.synchronize()
            for x, y in zip(a, b):
                assert bool(torch.isfinite(x).all())
                assert torch.equal(x[others], y[others]), (what, build)
    finally:
        m.close()
