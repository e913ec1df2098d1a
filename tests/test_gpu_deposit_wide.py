"""The deposit's larger workgroups and tiles (512 particles over 6144 cells)
against the oracle: where they are taken (the size rule is asked), with
particles as arrays in and out of the build's order and as records, for dense,
sparse and mixed spreads (workgroup tile, wavefront tiles, corner by corner),
a full and partly filled last workgroups, some particles outside, unequal edges
and cells that are no powers of two.  Tolerance: the worst rounding of a sum of
n like-signed terms in any order, (n + 16) 2^-53 of the largest cell."""
import ctypes as C

import numpy as np
import pytest

from oracle import oracle as O
from paper_1812_03689_amd import workloads as W
from test_gpu_deposit_paths import BOXES, draw

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N0 = (48, 40, 56)


@pytest.mark.parametrize("spread", ["dense", "sparse", "mixed"])
@pytest.mark.parametrize("n", [262144, 262145, 262144 + 513, 600001])
@pytest.mark.parametrize("pos", [np.float64, np.float32])
def test_wide_deposit_equals_oracle(n, spread, pos):
    print("wide deposit", n, spread, pos, flush=True)
    from paper_1812_03689_amd import amrmg as A
    rng = np.random.default_rng(n)
    p = draw(n, spread, rng).astype(pos)
    q = rng.random(n) + 0.5
    w = W.Workload("deposit", W.Particles(*(np.ascontiguousarray(p[:, d]) for d in range(3)), q), N0, 2, [], [], 1e-8,
                   explicit_boxes=BOXES, hi=(0.9, 0.9, 0.9))
    ctx = A.Context(A.make_params(w.n0, max_level=2, hi=w.hi))
    x, y, z, qd = (torch.as_tensor(a, device="cuda") for a in (*w.particles.__dict__.values(),))
    ctx.build_hierarchy(x, y, z, qd, explicit_boxes=BOXES)
    wide = A.lib()._Z9wide_tilePK9amrmg_ctxi  # bool wide_tile(const amrmg_ctx *, int level)
    wide.argtypes, wide.restype = [C.c_void_p, C.c_int], C.c_bool
    assert wide(ctx.h, 2)
    H = O.hierarchy_from_workload(w)
    want = H.deposit_all(W.Particles(*(a.astype(np.float64) for a in (w.particles.x, w.particles.y, w.particles.z)), q))
    inside = int(np.all((p.astype(np.float64) >= 0) & (p.astype(np.float64) < 0.9), axis=1).sum())

    def check(rho, nout, outside):
        assert nout == outside
        for r, o in zip(rho, want):
            assert np.abs(r.cpu().numpy() - o).max() <= (n + 16) * 2.0 ** -53 * max(np.abs(o).max(), 1e-300)

    check(*ctx.deposit_built(), n - inside)
    check(*ctx.deposit(x, y, z, qd), n - inside)
    # moved within the build's order, and another count: the caller's order
    check(*ctx.deposit(*(torch.flip(a, (0,)) for a in (x, y, z, qd))), n - inside)
    first = int(not np.all((p[0].astype(np.float64) >= 0) & (p[0].astype(np.float64) < 0.9)))
    more = [torch.cat([a, a[:1]]) for a in (x, y, z)]
    check(*ctx.deposit(*more, torch.cat([qd, torch.zeros_like(qd[:1])])), n - inside + first)
