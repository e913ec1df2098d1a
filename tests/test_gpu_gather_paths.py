"""The gather's ways through its kernels against the oracle's interpolation of
the same field: the caller's order (few particles), the visiting order, moved
particles read as records, the field through LDS (dense) and cell by cell
(sparse), stencils across box faces and between levels, particles outside;
arrays and ordered copy; cell sizes that are no powers of two.  Every way adds
the same products in the same order, so beside the oracle's round-off (eight
products: 16 2^-53 of the largest value) the ways agree bit for bit."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1812_03689_amd import workloads as W
from test_gpu_deposit_paths import BOXES, draw

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("spread", ["dense", "sparse", "mixed"])
@pytest.mark.parametrize("n", [1, 65, 65535, 65536, 524289, 800000])
@pytest.mark.parametrize("pos", [np.float64, np.float32])
def test_gather_equals_oracle(n, spread, pos):
    print("gather", n, spread, pos, flush=True)
    from paper_1812_03689_amd import amrmg as A
    rng = np.random.default_rng(n)
    p = draw(n, spread, rng).astype(pos)
    w = W.Workload("gather", W.Particles(*(np.ascontiguousarray(p[:, d]) for d in range(3)), np.ones(n)), (32, 32, 32),
                   2, [], [], 1e-8, explicit_boxes=BOXES, hi=(0.9, 0.9, 0.9))
    ctx = A.Context(A.make_params(w.n0, max_level=2, hi=w.hi))
    x, y, z, q = (torch.as_tensor(a, device="cuda") for a in (*w.particles.__dict__.values(),))
    # built on other positions, so that the gather's particles have moved
    ctx.build_hierarchy(*(torch.flip(a, (0,)) for a in (x, y, z)), q, explicit_boxes=BOXES)
    E = [torch.as_tensor(rng.standard_normal(c), device="cuda") for c in ctx.info["ncells"] for _ in range(3)]
    H = O.hierarchy_from_workload(w)
    want = H.gather(W.Particles(*(a.astype(np.float64) for a in (w.particles.x, w.particles.y, w.particles.z)),
                                w.particles.q), [t.cpu().numpy() for t in E])
    got = ctx.gather(x, y, z, E)
    for g, o in zip(got, want):
        assert np.abs(g.cpu().numpy() - o).max() <= 16 * 2.0 ** -53 * 8 * max(np.abs(o).max(), 1.0)
    built = ctx.gather_built(E)
    some = ctx.gather(*(torch.cat([a, a[:1]]) for a in (x, y, z)), E)  # another count: the caller's order
    for g, b, s in zip(got, built, some):
        assert torch.equal(g, torch.flip(b, (0,)))
        assert torch.equal(g, s[:n])
