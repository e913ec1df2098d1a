"""A wait that no run shows reliably, read from the machine code of the built
library: in k_level_norms every wavefront of a workgroup stores its sum, then
one thread counts the workgroup in, and the last workgroup counted reads all
sums.  Between a wavefront's store and the barrier before the count there must
be a wait for that store (the count's own ordering covers the counting
wavefront's stores alone; a barrier waits for none)."""
import os
import re
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    from paper_1812_03689_amd import build
    if not os.path.exists(build.LIB):
        build.build()
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    d = tmp_path_factory.mktemp("code")
    lib = os.path.join(str(d), "lib.so")
    os.symlink(build.LIB, lib)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=str(d), capture_output=True, check=True)
    text = ""
    for f in sorted(os.listdir(str(d))):
        if "gfx950" in f:
            text += subprocess.run([OBJDUMP, "-d", f], cwd=str(d), capture_output=True, check=True, text=True).stdout
    return text


def test_sums_arrive_before_the_count(code):
    m = re.search(r"^[0-9a-f]+ <\S*k_level_norms\S*>:\n(.*?)s_endpgm", code, re.S | re.M)
    assert m, "k_level_norms not found"
    ins = [l.split("//")[0].strip() for l in m.group(1).splitlines()]
    count = next(i for i, l in enumerate(ins) if l.startswith("global_atomic_add"))
    barrier = max(i for i in range(count) if ins[i].startswith("s_barrier"))
    store = max(i for i in range(barrier) if ins[i].startswith("global_store_dwordx2"))
    assert any(l.startswith("s_waitcnt") and "vmcnt(0)" in l for l in ins[store:barrier]), "\n".join(ins[store:count + 1])
