"""Calls that find no room on the device for buffers that only save time.  A
child process puts a function in front of hipMalloc that refuses chosen sizes
(tests/native/alloc_limit.c):

* no room for the particle records of a build: deposit and gather read the
  arrays, the same values as with records (the gather bit for bit, the deposit
  to the rounding of a sum of n like-signed terms in any order, (n + 16) 2^-53
  of the largest cell), dense particles and sparse ones;
* no room for a solve's workspace while records are kept: they are given back
  and the solve goes through; deposit and gather afterwards read the arrays;
* records that a capture has recorded are not given back: that solve is
  refused, and replays of the captured deposit still give the charge."""
import ctypes as C
import os
import subprocess
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BOXES = [(1, 16, 16, 16, 48, 48, 48)]
N = 700001


def arrays(spread):
    import torch
    rng = np.random.default_rng(3)
    p = 0.3 + 0.35 * rng.random((3, N)) if spread == "dense" else rng.random((3, N))
    return [torch.as_tensor(a, device="cuda") for a in (*p, rng.random(N) + 0.5)]


def context(max_level=1, stream=None):
    from paper_1812_03689_amd import amrmg as A
    return A.Context(A.make_params((32, 32, 32), max_level=max_level), stream=stream)


def load_limit(lib):
    """hipMalloc of every library loaded from here on goes through lib."""
    lim = C.CDLL(lib, mode=C.RTLD_GLOBAL)
    import torch
    from paper_1812_03689_amd import amrmg as A
    A.lib()
    torch.zeros(1)
    path, = {l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l}
    lim.alloc_limit_real.argtypes = [C.c_void_p]
    lim.alloc_limit_real(C.cast(C.CDLL(path).hipMalloc, C.c_void_p))
    lim.alloc_limit_arm.argtypes = [C.c_size_t, C.c_size_t, C.c_int]
    return lim


def arm(lim, need, count=1):
    # a buffer is allocated a quarter larger than asked for, and a page
    lim.alloc_limit_arm(need + need // 4 + 4096, need + need // 4 + 4097, count)


def same_charge(a, b):
    import torch
    for u, v in zip(a, b):
        assert float((u - v).abs().max()) <= (N + 16) * 2.0 ** -53 * float(v.abs().max())
    torch.cuda.synchronize()


def child_records(lim, spread):
    import torch
    x, y, z, q = arrays(spread)
    g = torch.Generator(device="cuda").manual_seed(1)
    out = []
    for refuse in (0, 1):
        ctx = context(0 if spread == "dense" else 1)
        arm(lim, 32 * N, refuse)
        ctx.build_hierarchy(x, y, z, q, explicit_boxes=BOXES if spread != "dense" else None)
        assert lim.alloc_limit_failed() == refuse
        g.manual_seed(1)
        E = [torch.randn(c, generator=g, device="cuda", dtype=torch.float64) for c in ctx.info["ncells"] for _ in range(3)]
        moved = [torch.flip(t, (0,)) for t in (x, y, z)]
        out.append((ctx.deposit_built()[0], ctx.deposit(*moved, q)[0], ctx.gather(*moved, E), ctx.gather_built(E)))
    for a, b in zip(out[0][:2], out[1][:2]):
        same_charge(b, a)
    for a, b in zip(out[0][2:], out[1][2:]):
        assert all(torch.equal(u, v) for u, v in zip(a, b))


def child_workspace(lim, _):
    import torch
    from paper_1812_03689_amd import amrmg as A
    x, y, z, q = arrays("dense")
    ctx = context()
    ctx.build_hierarchy(x, y, z, q, explicit_boxes=BOXES)
    rho, _ = ctx.deposit(x, y, z, q)
    need = A.amrmg_workspace_size(ctx.h)
    arm(lim, need)
    phi, E, st = ctx.solve(rho)
    assert lim.alloc_limit_failed() == 1 and st["converged"]
    got = ctx.gather(x, y, z, E)
    same_charge(ctx.deposit(x, y, z, q)[0], rho)
    ctx.build_hierarchy(x, y, z, q, explicit_boxes=BOXES)  # records again
    assert all(torch.equal(a, b) for a, b in zip(got, ctx.gather(x, y, z, E)))


def child_capture(lim, _):
    import torch
    from paper_1812_03689_amd import amrmg as A
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        x, y, z, q = arrays("dense")
        ctx = context(stream=s)
        ctx.build_hierarchy(x, y, z, q, explicit_boxes=BOXES)
        want, _ = ctx.deposit(x, y, z, q)
        rho = ctx.level_arrays()
        P = A._ptrs(rho)
        s.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            rc = A.lib().amrmg_deposit(ctx.h, A.AMRMG_POS_F64, *(C.c_void_p(t.data_ptr()) for t in (x, y, z, q)),
                                       C.c_int64(N), P, None)
        assert rc == A.AMRMG_OK
        need = A.amrmg_workspace_size(ctx.h)
        arm(lim, need)
        with pytest.raises(A.AmrmgError) as e:
            ctx.solve(want)
        assert e.value.status == A.AMRMG_E_OOM
        for _ in range(3):
            for t in rho:
                t.fill_(7.0)
            graph.replay()
            s.synchronize()
            same_charge(rho, want)
            assert ctx.solve(want)[2]["converged"]
        ctx.build_hierarchy(x, y, z, q, explicit_boxes=BOXES)


@pytest.fixture(scope="module")
def limit(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("limit") / "alloc_limit.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", os.path.join(ROOT, "tests", "native", "alloc_limit.c"), "-o", so],
                   check=True)
    return so


@pytest.mark.parametrize("what,arg", [("records", "dense"), ("records", "sparse"), ("workspace", "-"), ("capture", "-")])
def test_no_room(limit, what, arg):
    print("no room", what, arg, flush=True)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), limit, what, arg], cwd=ROOT, capture_output=True,
                       text=True, timeout=110, env=dict(os.environ, PYTHONPATH=ROOT))
    print(r.stdout[-2000:], r.stderr[-4000:], flush=True)
    assert r.returncode == 0 and "child ok" in r.stdout


if __name__ == "__main__":
    limit_lib = load_limit(sys.argv[1])
    globals()["child_" + sys.argv[2]](limit_lib, sys.argv[3])
    print("child ok", flush=True)
