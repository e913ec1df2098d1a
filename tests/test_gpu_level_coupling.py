"""What a finer level reads of the coarser one's correction: parents and the
windows of the coarse-fine ghosts.  The last post-smoothing sweep stores only
those bricks, so every brick of the coarser level that the tables name must be
marked: the solve of meshes whose fine boxes lie one to five coarse cells from
brick faces, along edges and corners, with an odd and an even number of post-
smoothing sweeps, from two different amounts of garbage in the workspace,
gives the same phi bit for bit (no charge: no atomics, one order of every sum)
and meets its tolerance by the residual of the operator itself."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

MESHES = [
    [(1, 16, 16, 16, 40, 48, 32)],
    [(1, 16, 16, 16, 32, 32, 32), (1, 32, 32, 32, 48, 48, 56), (1, 32, 16, 16, 40, 32, 24)],
    [(1, 0, 8, 40, 24, 72, 80), (1, 24, 24, 40, 80, 40, 72)],
    [(1, 16, 16, 16, 64, 64, 64), (2, 40, 40, 40, 56, 64, 72), (2, 56, 48, 48, 88, 56, 88), (2, 88, 56, 56, 96, 96, 64)],
]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("nu2", [1, 3, 4])
@pytest.mark.parametrize("mesh", range(len(MESHES)))
def test_unread_bricks_do_not_matter(mesh, nu2, precision):
    from paper_1812_03689_amd import amrmg as A
    print("coupling", mesh, nu2, precision, flush=True)
    n0 = (40, 40, 40)
    ctx = A.Context(A.make_params(n0, max_level=MESHES[mesh][-1][0], precision=precision, nu2=nu2, max_iters=80,
                                  monopoles=[(1.0, 0.41, 0.52, 0.47)]))
    e = torch.zeros(0, dtype=torch.float64, device="cuda")
    ctx.build_hierarchy(e, e, e, e, explicit_boxes=MESHES[mesh])
    gen = torch.Generator(device="cuda").manual_seed(mesh)
    rho = [torch.randn(n, generator=gen, device="cuda", dtype=torch.float64) for n in ctx.info["ncells"]]
    need = A.amrmg_workspace_size(ctx.h)
    got = []
    for fill in (0, 0x7f):  # zeros, and NaN / huge values
        ws = torch.full((need + 256,), fill, dtype=torch.uint8, device="cuda")
        ws = ws[(-ws.data_ptr()) % 256:][:need]
        A.amrmg_set_workspace(ctx.h, ws)
        phi, _, st = ctx.solve(rho, tol=1e-9, want_E=False)
        assert st["converged"]
        got.append(phi)
    for a, b in zip(*got):
        assert torch.equal(a, b)
    r, b = ctx.residual(rho, got[0]), ctx.residual(rho, [torch.zeros_like(t) for t in rho])
    for u, v in zip(r, b):
        assert float(u.norm()) <= 1.0001e-9 * float(v.norm())
