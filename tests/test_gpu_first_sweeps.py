"""The fused first two sweeps against sweeps that are launched one by one: with
nu1 = 1, 2, 3 and 4 pre-smoothing sweeps (one sweep: the zero-start kernel
alone; from two on the fused kernel) every cycle solves the same composite
problem, so the FP64 solutions agree to the tolerance's error on meshes with
refinement at the domain's edge, coarse-fine faces on every side, a Robin
boundary and an odd number of bricks per row; and the fused kernel's cycle
converges as two separate sweeps do: not slower than one sweep, not more than
one cycle apart from three."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

MESHES = [
    ((32, 32, 32), [(1, 16, 16, 16, 48, 48, 48)]),
    ((40, 24, 56), [(1, 0, 0, 0, 24, 16, 32), (1, 24, 16, 32, 56, 40, 72), (2, 64, 48, 80, 96, 64, 112)]),
    ((72, 64, 80), [(1, 40, 40, 40, 104, 72, 120), (2, 96, 96, 96, 128, 128, 160)]),
]


def run(n0, boxes, nu1, robin, precision, g):
    from paper_1812_03689_amd import amrmg as A
    h = 1.0 / max(n0)
    ctx = A.Context(A.make_params(n0, max_level=boxes[-1][0], precision=precision, nu1=nu1, hi=tuple(v * h for v in n0),
                                  robin_d=robin, max_grid_size=64))
    e = torch.zeros(0, dtype=torch.float64, device="cuda")
    ctx.build_hierarchy(e, e, e, e, explicit_boxes=boxes)
    gen = torch.Generator(device="cuda").manual_seed(g)
    rho = [torch.randn(n, generator=gen, device="cuda", dtype=torch.float64) for n in ctx.info["ncells"]]
    phi, _, st = ctx.solve(rho, tol=1e-11, want_E=False)
    assert st["converged"]
    return phi, st["iters"]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("robin", [0.0, 1.7])
@pytest.mark.parametrize("mesh", range(len(MESHES)))
def test_same_solution(mesh, robin, precision):
    n0, boxes = MESHES[mesh]
    print("first sweeps", n0, robin, precision, flush=True)
    got = {nu1: run(n0, boxes, nu1, robin, precision, mesh) for nu1 in (1, 2, 3, 4)}
    ref, it1 = got[1]
    for nu1 in (2, 3, 4):
        phi, it = got[nu1]
        # a residual of 1e-11 leaves an error below the condition number (2 n / pi)^2 <= 3e4 times it
        for a, b in zip(phi, ref):
            assert float((a - b).norm() / b.norm()) <= 3e-7
        assert it <= it1
    assert got[2][1] <= got[3][1] + 2
