"""The build's paths by size, where they change: the visiting order at 127, 128
and 129 radix tiles (up to 128 every scatter workgroup sums the tiles'
histograms itself; 9- and 10-bit digits) is NumPy's stable argsort of the same
keys, element by element; and the tagged boxes of level 1, from the marks that
the kernel writes to host memory (60 blocks, a part of a word, to 270,000),
cover exactly the blocks that the kept charge of level 0, tagged and dilated
here, marks."""
import numpy as np
import pytest

from test_gpu_visiting_order import build, morton_keys
from paper_1812_03689_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TILE = 1024


@pytest.mark.parametrize("n0", [(16, 16, 16), (64, 64, 64), (1000, 16, 24)])
@pytest.mark.parametrize("n", [127 * TILE + 1, 128 * TILE, 128 * TILE + 1])
def test_order_around_the_tile_limit(n, n0):
    p = W.gaussian_bunch(n, sigma=(0.05, 0.05, 0.1), seed=W.seed_for(3, n % 89))
    ctx, (x, y, z) = build(p, n0, 1)
    perm = ctx.visiting_order().cpu().numpy()
    keys = morton_keys(*(t.cpu().numpy() for t in (x, y, z)), (0, 0, 0), (1, 1, 1), n0, 1)
    assert np.array_equal(perm, np.argsort(keys, kind="stable"))


@pytest.mark.parametrize("n0", [(24, 16, 40), (256, 256, 256), (264, 256, 256)])
def test_tagged_blocks(n0):
    p = W.gaussian_bunch(50000, sigma=(0.05, 0.07, 0.1), seed=W.seed_for(3, 5))
    ctx, _ = build(p, n0, 1, tag=0.2)
    rho, _ = ctx.deposit_built()
    v = rho[0].cpu().numpy().reshape(n0[::-1])  # [z, y, x]
    tag = np.abs(v) > 0.2 * np.abs(v).max()
    nbuf, half = ctx.params.n_buffer, ctx.params.blocking_factor // 2
    want = np.zeros([m // half for m in n0[::-1]], dtype=bool)
    for k, j, i in np.argwhere(tag):
        s = tuple(slice(max(0, c - nbuf) // half, min(m - 1, c + nbuf) // half + 1) for c, m in zip((k, j, i), n0[::-1]))
        want[s] = True
    assert want.any()
    got = np.zeros_like(want, dtype=int)
    bf = ctx.params.blocking_factor
    for b in ctx.boxes(1)[0]:
        got[b[2] // bf:b[5] // bf, b[1] // bf:b[4] // bf, b[0] // bf:b[3] // bf] += 1
    assert np.array_equal(got, want.astype(int))
