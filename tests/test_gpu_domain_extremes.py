"""Charge and field interpolation in domains whose cell size or its reciprocal
is no ordinary number (subnormal cells, a domain whose extent overflows): the
stencil position (x - lo) / h - 1/2 is the true quotient's there too.  The
gathered field is the interpolation written out in NumPy, to the rounding of
eight products and their weights (32 2^-53 of the largest value; the position
is the same bits), and finite; the charge lands in the same cells."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

DOMAINS = [(0.0, 1e-310), (-3e-309, 5e-309), (0.0, 1.6e-307), (-1e308, 1e308), (0.0, 1.7e308), (0.0, 1e-200), (0.0, 1e200)]


def interpolate(x, lo, hi, n, F):
    i, f = [], []
    for d in range(3):
        with np.errstate(over="ignore"):
            h = (np.float64(hi) - np.float64(lo)) / n
        s = (x[d] - lo) / h - 0.5
        a = np.floor(s)
        f.append(s - a)
        i.append([np.clip(a.astype(np.int64) + k, 0, n - 1) for k in (0, 1)])
    out = np.zeros(x[0].size)
    for c in range(8):
        b = [(c >> d) & 1 for d in range(3)]
        w = np.prod([f[d] if b[d] else 1.0 - f[d] for d in range(3)], axis=0)
        out += w * F[i[2][b[2]], i[1][b[1]], i[0][b[0]]]
    return out, [i[d][0] for d in range(3)]


@pytest.mark.parametrize("npart", [5000, 70001])
@pytest.mark.parametrize("lo,hi", DOMAINS)
def test_gather_and_deposit(lo, hi, npart):
    from paper_1812_03689_amd import amrmg as A
    print("domain", lo, hi, npart, flush=True)
    n = 16
    rng = np.random.default_rng(npart)
    ctx = A.Context(A.make_params((n, n, n), max_level=0, lo=(lo,) * 3, hi=(hi,) * 3))
    # (x - lo itself stays finite: at most 1.7e308)
    x = [np.clip(lo * (1.0 - t) + hi * t, lo, min(np.nextafter(hi, lo), lo / 2 + 1.2e308)) for t in rng.random((3, npart))]
    x[0][0] = lo
    dev = [torch.as_tensor(a, device="cuda") for a in x]
    q = torch.as_tensor(rng.random(npart) + 0.5, device="cuda")
    ctx.build_hierarchy(*dev, q)
    F = rng.standard_normal((3, n, n, n))
    got = ctx.gather(*dev, [torch.as_tensor(F[d].reshape(-1), device="cuda") for d in range(3)])
    for d in range(3):
        want, low = interpolate(x, lo, hi, n, F[d])
        assert np.isfinite(want).all()
        assert np.abs(got[d].cpu().numpy() - want).max() <= 32 * 2.0 ** -53 * np.abs(F[d]).max()
    # which cells hold charge: the value itself leaves the range with the cell's volume
    rho, nout = ctx.deposit(*dev, q)
    assert nout == 0
    hit = np.zeros((n, n, n), dtype=bool)
    for c in range(8):
        b = [(c >> d) & 1 for d in range(3)]
        hit[tuple(np.minimum(low[d] + b[d], n - 1) for d in (2, 1, 0))] = True
    r = rho[0].cpu().numpy().reshape(n, n, n)
    with np.errstate(over="ignore", divide="ignore"):
        h = (np.float64(hi) - np.float64(lo)) / n
        if 1.0 / (h * h * h) > 0.0:  # (a huge cell's density is zero)
            assert not (r[~hit] != 0.0).any()
