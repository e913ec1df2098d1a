"""The level norms' ways through their kernel: one workgroup (few pieces of 512
bricks, an uneven last one) and several (more than 64 pieces, counted in by
the last), the norms of the residual and of the right-hand side in one launch,
all three norms.  The norms a solve reports after no useful cycle are those of
the residual kernel's own output: rel_residual = |r| / |b| with r, b from
amrmg_residual at the returned phi and at phi = 0, to the rounding of a sum of
n non-negative terms in any order, n 2^-53."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("norm_p", [0, 1, 2])
@pytest.mark.parametrize("n0", [(8, 8, 8), (72, 64, 56), (256, 256, 288)])
def test_reported_norms(n0, norm_p):
    from paper_1812_03689_amd import amrmg as A
    print("norms", n0, norm_p, flush=True)
    h = 1.0 / max(n0)
    mid = tuple(0.5 * v * h for v in n0)
    ctx = A.Context(A.make_params(n0, max_level=0, precision="fp64", norm_p=norm_p, max_iters=1, bottom="auto",
                                  hi=tuple(v * h for v in n0), monopoles=[(1.0,) + mid]))
    e = torch.zeros(0, dtype=torch.float64, device="cuda")
    ctx.build_hierarchy(e, e, e, e)
    g = torch.Generator(device="cuda").manual_seed(norm_p)
    rho = [torch.randn(n, generator=g, device="cuda", dtype=torch.float64) for n in ctx.info["ncells"]]
    phi = [0.1 * torch.randn(n, generator=g, device="cuda", dtype=torch.float64) for n in ctx.info["ncells"]]

    def norm(v):
        v = v.cpu().numpy()
        return np.abs(v).max() if norm_p == 0 else np.linalg.norm(v, norm_p)

    b = ctx.residual(rho, [torch.zeros_like(t) for t in phi])
    phi, _, st = ctx.solve(rho, phi=phi, tol=1e-300, want_E=False)
    r = ctx.residual(rho, phi)
    n = sum(ctx.info["ncells"])
    for l, rel in enumerate(st["rel_residual"]):
        want = norm(r[l]) / norm(b[l])
        # the residual itself is evaluated twice from the same phi by one kernel
        assert abs(rel - want) <= (n + 8) * 2.0 ** -53 * want
