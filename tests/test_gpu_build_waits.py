"""A build that uploads the direct solve's tables (a new context, other edges)
waits for its stream no more often than one that finds them on the device.  A
child process counts the waits (tests/native/count_waits.c)."""
import ctypes as C
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def child(so):
    count = C.CDLL(so, mode=C.RTLD_GLOBAL)
    import torch
    from paper_1812_03689_amd import amrmg as A
    A.lib()
    path, = {l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l}
    count.count_waits_real.argtypes = [C.c_void_p]
    count.count_waits_real(C.cast(C.CDLL(path).hipStreamSynchronize, C.c_void_p))
    e = torch.zeros(0, dtype=torch.float64, device="cuda")
    for n in (32, 40):
        ctx = A.Context(A.make_params((n, n, n), max_level=1))
        waits = []
        for _ in range(3):
            before = count.count_waits()
            ctx.build_hierarchy(e, e, e, e, explicit_boxes=[(1, 16, 16, 16, 32, 32, 32)])
            waits.append(count.count_waits() - before)
        print(n, waits, flush=True)
        assert waits[0] == waits[1] == waits[2] > 0
        # the tables are the right ones
        g = torch.Generator(device="cuda").manual_seed(n)
        rho = [torch.randn(c, generator=g, device="cuda", dtype=torch.float64) for c in ctx.info["ncells"]]
        assert ctx.solve(rho, tol=1e-9)[2]["iters"] <= 14


def test_waits_of_a_new_context(tmp_path):
    so = str(tmp_path / "count_waits.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", os.path.join(ROOT, "tests", "native", "count_waits.c"), "-o", so],
                   check=True)
    print("build waits", flush=True)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), so], cwd=ROOT, capture_output=True, text=True,
                       timeout=110, env=dict(os.environ, PYTHONPATH=ROOT))
    print(r.stdout[-2000:], r.stderr[-4000:], flush=True)
    assert r.returncode == 0 and "child ok" in r.stdout


if __name__ == "__main__":
    child(sys.argv[1])
    print("child ok", flush=True)
