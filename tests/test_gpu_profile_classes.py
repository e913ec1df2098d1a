"""The deposit and gather classes hold every launch that reads the particles: a
deposit or gather of moved particles that packs records first (from 524288
particles, in the build's order) records two launches with the bytes of one,
smaller ones and the built particles' one."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("pos", [torch.float64, torch.float32])
@pytest.mark.parametrize("n,launches", [(524288, 2), (524287, 1), (5000, 1)])
def test_packing_is_counted(n, launches, pos):
    from paper_1812_03689_amd import amrmg as A
    print("profile classes", n, pos, flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    x, y, z = (torch.rand(n, generator=g, device="cuda", dtype=pos) for _ in range(3))
    q = torch.ones(n, device="cuda", dtype=torch.float64)
    ctx = A.Context(A.make_params((32, 32, 32), max_level=0))
    ctx.build_hierarchy(x, y, z, q)
    E = ctx.level_arrays(3)
    w = 4 if pos == torch.float32 else 8
    bytes_of = {"deposit": n * (3.0 * w + 8.0) + 8.0 * 32 ** 3, "gather": n * (3.0 * w + 24.0)}
    A.amrmg_profile_enable(ctx.h, ["deposit", "gather"])
    ctx.deposit(x, y, z, q)
    ctx.gather(x, y, z, E)
    for c, want in bytes_of.items():
        ms, by = A.amrmg_profile_launches(ctx.h, c)
        tot = A.amrmg_profile_read(ctx.h, c)
        assert len(ms) == tot["launches"] == launches and (ms > 0.0).all()
        assert tot["bytes"] == by.sum() == want
    A.amrmg_profile_enable(ctx.h, ["deposit"])
    ctx.deposit_built()
    assert A.amrmg_profile_read(ctx.h, "deposit")["launches"] == 1
