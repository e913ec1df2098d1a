"""The deposit's ways through its kernel against the oracle, at the sizes
where they change: a workgroup's tile (dense particles), a wavefront's tile
and corner by corner (sparse ones), partly filled wavefronts and workgroups,
both workgroup sizes, particles read as arrays and as records, in and out of
the build's order, some outside the domain; cell sizes that are no powers of
two.  Tolerance: the worst rounding of a sum of n like-signed terms in any
order, (n + 16) 2^-53 of the largest cell."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1812_03689_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

BOXES = [(1, 8, 8, 8, 40, 40, 24), (1, 8, 8, 24, 40, 40, 56), (2, 32, 32, 32, 64, 64, 64), (2, 64, 32, 32, 72, 64, 64)]


def draw(n, spread, rng):
    """n points around the middle of [0, 0.9)^3: all within a cell ("dense"), over
    the whole domain ("sparse"), or both with a few outside ("mixed")."""
    dense = 0.41 + 0.003 * rng.random((n, 3))
    sparse = 0.9 * rng.random((n, 3))
    if spread == "dense":
        return dense
    if spread == "sparse":
        return sparse
    p = np.where((np.arange(n) % 3 == 0)[:, None], dense, sparse)
    p[::97] += 1.0
    return p


@pytest.mark.parametrize("spread", ["dense", "sparse", "mixed"])
@pytest.mark.parametrize("n", [1, 64, 257, 5000, 262145, 524289])
@pytest.mark.parametrize("pos", [np.float64, np.float32])
def test_deposit_equals_oracle(n, spread, pos):
    print("deposit", n, spread, pos, flush=True)
    from paper_1812_03689_amd import amrmg as A
    rng = np.random.default_rng(n)
    p = draw(n, spread, rng).astype(pos)
    q = rng.random(n) + 0.5
    w = W.Workload("deposit", W.Particles(*(np.ascontiguousarray(p[:, d]) for d in range(3)), q), (32, 32, 32), 2, [],
                   [], 1e-8, explicit_boxes=BOXES, hi=(0.9, 0.9, 0.9))
    ctx = A.Context(A.make_params(w.n0, max_level=2, hi=w.hi))
    x, y, z, qd = (torch.as_tensor(a, device="cuda") for a in (*w.particles.__dict__.values(),))
    ctx.build_hierarchy(x, y, z, qd, explicit_boxes=BOXES)
    H = O.hierarchy_from_workload(w)
    want = H.deposit_all(W.Particles(*(a.astype(np.float64) for a in (w.particles.x, w.particles.y, w.particles.z)), q))
    inside = int(np.all((p.astype(np.float64) >= 0) & (p.astype(np.float64) < 0.9), axis=1).sum())

    def check(rho, nout, scale=1.0):
        assert nout == n - inside
        for r, o in zip(rho, want):
            tol = (n + 16) * 2.0 ** -53 * max(np.abs(o).max(), 1e-300)
            assert np.abs(r.cpu().numpy() - scale * o).max() <= tol

    check(*ctx.deposit_built())
    check(*ctx.deposit(x, y, z, qd))
    # another count than the build's: visited in the caller's order
    if n <= 5000:
        zero = torch.zeros(1, dtype=torch.float64, device="cuda")
        rho, nout = ctx.deposit(*(torch.cat([a, a[:1]]) for a in (x, y, z)), torch.cat([qd, zero]))
        outside = int(not np.all((p[0].astype(np.float64) >= 0) & (p[0].astype(np.float64) < 0.9)))
        check(rho, nout - outside)
