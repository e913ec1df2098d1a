"""The direct solve of the coarsest grid at the edges of its 16-wide matrix
tiles and operand sizes (32, 64, 128): one level that is the coarsest grid
itself, so that one cycle solves the discrete problem; phi against the sine
diagonalisation in NumPy FP64, for FP64 and FP32 cycles and for a batch of
all.  Tolerance: the transforms' rounding, condition number ~ (2 n / pi)^2
below 7e3 times 1e-16, far below 1e-11; the mixed cycle stops at 1e-10."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

EDGES = [(8, 8, 8), (16, 24, 8), (32, 16, 40), (40, 32, 24), (64, 48, 16), (72, 64, 56), (88, 72, 120), (128, 112, 104)]


def solved(rho, n, h):
    """The homogeneous Dirichlet problem -L phi = rho by its sine vectors."""
    b = rho.reshape(n[::-1])
    lam = []
    for d in range(3):
        k = np.arange(n[d])
        S = np.sin(np.pi * (k[:, None] + 1) * (k[None, :] + 0.5) / n[d])
        S /= np.linalg.norm(S, axis=1, keepdims=True)
        lam.append((S, 4 * np.sin(np.pi * (k + 1) / (2 * n[d])) ** 2 / h ** 2))
    for d in range(3):
        b = np.moveaxis(np.tensordot(lam[d][0], np.moveaxis(b, 2 - d, 0), 1), 0, 2 - d)
    b = b / (lam[2][1][:, None, None] + lam[1][1][None, :, None] + lam[0][1][None, None, :])
    for d in range(3):
        b = np.moveaxis(np.tensordot(lam[d][0].T, np.moveaxis(b, 2 - d, 0), 1), 0, 2 - d)
    return b.reshape(-1)


def problem(n, precision):
    from paper_1812_03689_amd import amrmg as A
    h = 1.0 / max(n)
    ctx = A.Context(A.make_params(n, max_level=0, precision=precision, hi=tuple(v * h for v in n)))
    e = torch.zeros(0, dtype=torch.float64, device="cuda")
    ctx.build_hierarchy(e, e, e, e)
    rho = np.random.default_rng(sum(n)).standard_normal(n[0] * n[1] * n[2])
    return ctx, rho, solved(rho, n, h)


def close(phi, want, tol=1e-10):
    return np.linalg.norm(phi[0].cpu().numpy() - want) <= tol * np.linalg.norm(want)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n", EDGES)
def test_one_level(n, precision):
    print("direct", n, precision, flush=True)
    ctx, rho, want = problem(n, precision)
    phi, _, st = ctx.solve([torch.as_tensor(rho, device="cuda")], tol=1e-10)
    assert st["converged"] and close(phi, want)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_batch_of_all(precision):
    from paper_1812_03689_amd import amrmg as A
    print("direct batch", precision, flush=True)
    ps = [problem(n, precision) for n in EDGES]
    phi = [c.level_arrays() for c, _, _ in ps]
    A.amrmg_solve_batch([c.h for c, _, _ in ps], [[torch.as_tensor(r, device="cuda")] for _, r, _ in ps], phi, 1e-10)
    for u, (_, _, want) in zip(phi, ps):
        assert close(u, want)
