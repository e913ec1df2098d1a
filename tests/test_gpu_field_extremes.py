"""E of potentials at the ends of the number range: quotients that overflow,
infinities, differences of infinities and subnormal values come out as the
division -(u+ - u-) / (2 h) gives them in NumPy, value by value (the kernel
does these same operations, so no tolerance; Dirichlet ghosts of zero data
are -u, exact).  No iteration runs (max_iters = 0), so that the field is that
of the potential handed in, and a level of more than 16384 bricks takes the
kernel's other workgroup size."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def extremes(n, rng):
    v = rng.standard_normal(n) * 10.0 ** rng.integers(-320, 308, n)
    v[rng.random(n) < 0.05] = np.inf
    v[rng.random(n) < 0.05] = -np.inf
    v[rng.random(n) < 0.05] = 1.7e308
    v[rng.random(n) < 0.05] = 0.0
    return v


@pytest.mark.parametrize("edge", [1.0, 1e-3, 7e3])
@pytest.mark.parametrize("n0", [(16, 24, 8), (208, 208, 208)])
def test_field_is_the_quotient(n0, edge):
    from paper_1812_03689_amd import amrmg as A
    print("field extremes", n0, edge, flush=True)
    hi = tuple(edge * v / max(n0) for v in n0)
    ctx = A.Context(A.make_params(n0, max_level=0, precision="fp64", max_iters=0, hi=hi))
    e = torch.zeros(0, dtype=torch.float64, device="cuda")
    ctx.build_hierarchy(e, e, e, e)
    u = extremes(n0[0] * n0[1] * n0[2], np.random.default_rng(n0[0]))
    rho = [torch.zeros(u.size, dtype=torch.float64, device="cuda")]
    phi, E, _ = ctx.solve(rho, phi=[torch.as_tensor(u, device="cuda")], tol=1e-8)
    assert np.array_equal(phi[0].cpu().numpy(), u)
    w = u.reshape(n0[::-1])  # [z, y, x]
    for d in range(3):
        m = np.moveaxis(w, 2 - d, 0)
        p = np.concatenate([-m[:1], m, -m[-1:]])
        with np.errstate(all="ignore"):
            want = np.moveaxis(-(p[2:] - p[:-2]) / (2.0 * ((hi[d] - 0.0) / n0[d])), 0, 2 - d)
        got = E[d].cpu().numpy().reshape(w.shape)
        assert np.isinf(want).any() and np.isnan(want).any()
        assert np.array_equal(got, want, equal_nan=True)
