"""The first two sweeps in one launch against the same two launched one by one
(the zero-start sweep, then a plain one), e and the fine sums brick by brick on
every level: neighbours at the domain's edge (Dirichlet and Robin), coarse-fine
faces on every side and at their edges, one, two and four bricks a workgroup
(x-neighbours inside and outside it, a last workgroup that is not full), both
precisions.

Tolerance: a colour pass sums r / D and six weighted neighbours, whose weights
add up to at most one, in at most 16 roundings of terms that add up to at most
2 S, S = max |e| + 1.5 max |r| / D; an earlier pass's error comes in with weight
at most one.  Four passes, two ways of compiling them: 2 (4 (16 (2 S))) = 256
roundings of S.  A fine sum adds four cells of weight 1/3 and four of 1/5."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from test_gpu_first_sweeps import MESHES

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1812_03689_amd")


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    from paper_1812_03689_amd import amrmg as A
    so = str(tmp_path_factory.mktemp("shim") / "sweep_shim.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(PKG, "csrc"), "-isystem",
                    "/opt/rocm/include", os.path.join(ROOT, "tests", "native", "sweep_shim.cpp"), "-L" + PKG,
                    "-l:libamrmg.so", "-Wl,-rpath," + PKG, "-o", so], check=True)
    A.lib()
    L = C.CDLL(so)
    vp, i = C.c_void_p, C.c_int
    L.shim_fused.argtypes = [vp, i, i, i, vp, vp, vp, i, i]
    L.shim_separate.argtypes = [vp, i, i, i, vp, vp, vp, vp, vp, i, i]
    L.shim_fused.restype = L.shim_separate.restype = None
    return L


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("robin", [0.0, 1.7])
@pytest.mark.parametrize("mesh", range(len(MESHES)))
def test_fused_is_the_two_sweeps(shim, mesh, robin, f32):
    from paper_1812_03689_amd import amrmg as A
    n0, boxes = MESHES[mesh]
    print("pinned sweeps", n0, robin, f32, flush=True)
    edge = 1.0 / max(n0)
    ctx = A.Context(A.make_params(n0, max_level=boxes[-1][0], hi=tuple(v * edge for v in n0), robin_d=robin,
                                  max_grid_size=64))
    none = torch.zeros(0, dtype=torch.float64, device="cuda")
    ctx.build_hierarchy(none, none, none, none, explicit_boxes=boxes)
    t = A.amrmg_brick_tables(ctx.h)
    nb, dt = t["nbrick"], torch.float32 if f32 else torch.float64
    below = int(t["org"][:, 3].max()) + 1 - len(ctx.info["ncells"])  # levels below level 0
    g = torch.Generator(device="cuda").manual_seed(mesh)
    r = torch.randn(nb * 512, generator=g, device="cuda", dtype=dt)
    kinds = t["nbr"] < -t["nbc"]  # coarse-fine faces
    assert kinds[t["org"][:, 3] > below].any()
    for level in range(int(t["org"][:, 3].max()) + 1):
        ids = np.flatnonzero(t["org"][:, 3] == level)
        b0, n = int(ids[0]), len(ids)
        assert ids[-1] == b0 + n - 1
        h = edge * 2.0 ** (below - level)
        D = 6.0 / h ** 2
        for nt in (64, 128, 256):
            for faces in (0, 1):
                e = [torch.full_like(r, 3.0) for _ in range(2)]
                ffs = [torch.full((nb * 96,), 5.0, device="cuda", dtype=torch.float64) for _ in range(3)]
                tmp = torch.empty_like(r)
                torch.cuda.synchronize()
                shim.shim_fused(ctx.h, int(f32), b0, n, e[0].data_ptr(), r.data_ptr(), ffs[0].data_ptr(), faces, nt)
                shim.shim_separate(ctx.h, int(f32), b0, n, e[1].data_ptr(), tmp.data_ptr(), r.data_ptr(),
                                   ffs[1].data_ptr(), ffs[2].data_ptr(), faces, nt)
                torch.cuda.synchronize()
                lo, hi = b0 * 512, (b0 + n) * 512
                for a in e:  # nothing outside the level
                    assert bool((a[:lo] == 3.0).all()) and bool((a[hi:] == 3.0).all())
                S = float(e[1][lo:hi].abs().max()) + 1.5 * float(r[lo:hi].abs().max()) / D
                tol = 256 * (2.0 ** -24 if f32 else 2.0 ** -53) * S
                d = (e[0] - e[1])[lo:hi].abs().view(n, 512).amax(1)
                worst = int(d.argmax())
                assert float(d[worst]) <= tol, (level, nt, faces, b0 + worst, t["nbr"][b0 + worst], float(d[worst]), tol)
                if not faces:
                    assert bool((ffs[0] == 5.0).all())
                    continue
                assert torch.equal(ffs[0] == 5.0, ffs[1] == 5.0)
                assert bool(((ffs[0] != 5.0).view(nb, 6, 16).all(2).cpu() == torch.as_tensor(
                    kinds & (t["org"][:, 3:] == level))).all())
                assert float((ffs[0] - ffs[1]).abs().max()) <= 4 * (1.0 / 3.0 + 0.2) * tol + 16 * 2.0 ** -53 * S
