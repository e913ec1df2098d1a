"""A batch that finds no room beside the buffers that earlier batches left in
its first context: they are freed and it goes through, with the phi of a batch
in fresh contexts, bit for bit (the same kernels on the same merged tables).
A child process refuses the batch's first large allocation
(tests/native/alloc_limit.c)."""
import os
import subprocess
import sys

import pytest

from test_gpu_no_room import ROOT, limit, load_limit  # noqa: F401

pytestmark = pytest.mark.gpu


def problems(edges):
    import torch
    from paper_1812_03689_amd import amrmg as A
    e = torch.zeros(0, dtype=torch.float64, device="cuda")
    out = []
    for n in edges:
        ctx = A.Context(A.make_params((n, n, n), max_level=1))
        ctx.build_hierarchy(e, e, e, e, explicit_boxes=[(1, n // 2, n // 2, n // 2, n, n, n)])
        g = torch.Generator(device="cuda").manual_seed(n)
        out.append((ctx, [torch.randn(c, generator=g, device="cuda", dtype=torch.float64) for c in ctx.info["ncells"]]))
    return out


def solve(ps):
    from paper_1812_03689_amd import amrmg as A
    phi = [c.level_arrays() for c, _ in ps]
    st = A.amrmg_solve_batch([c.h for c, _ in ps], [r for _, r in ps], phi, 1e-9)
    assert all(s["converged"] for s in st)
    return phi


def child(lim):
    import torch
    want = solve(problems([16, 48, 32, 64]))
    ps = problems([16, 48, 32, 64])
    solve(ps[:2])
    lim.alloc_limit_arm(1 << 20, 1 << 40, 1)
    got = solve(ps)
    assert lim.alloc_limit_failed() == 1
    for a, b in zip(got, want):
        assert all(torch.equal(u, v) for u, v in zip(a, b))
    solve(ps[:2])


def test_batch_without_room(limit):  # noqa: F811
    print("batch without room", flush=True)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), limit], cwd=ROOT, capture_output=True, text=True,
                       timeout=110, env=dict(os.environ, PYTHONPATH=ROOT))
    print(r.stdout[-2000:], r.stderr[-4000:], flush=True)
    assert r.returncode == 0 and "child ok" in r.stdout


if __name__ == "__main__":
    child(load_limit(sys.argv[1]))
    print("child ok", flush=True)
