"""Nothing in the library's sources is out of reach: every launcher that
amrmg_kernels.hpp declares is called (its declaration, definition and
instantiation apart), and every kernel, device function and accessor of the
.hip files is named somewhere beside its definition."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1812_03689_amd", "csrc")


def sources():
    out = {}
    for p in glob.glob(os.path.join(CSRC, "*")):
        if p.endswith((".hip", ".cpp", ".hpp")):
            t = re.sub(r"/\*.*?\*/", " ", open(p).read(), flags=re.S)
            out[os.path.basename(p)] = re.sub(r"//[^\n]*", "", t)
    return out


def test_launchers_are_called():
    src = sources()
    names = set(re.findall(r"\b(launch_\w+)\s*\(", src["amrmg_kernels.hpp"]))
    assert len(names) > 20
    rest = "\n".join(t for f, t in src.items() if f != "amrmg_kernels.hpp")
    rest = re.sub(r"template void [^;]*;", "", rest)  # instantiations
    rest = re.sub(r"^(?:void|bool|hipError_t) launch_\w+\(", "", rest, flags=re.M)  # definitions
    unused = sorted(n for n in names if not re.search(r"\b%s\b" % n, rest))
    assert not unused, unused


def test_kernels_and_accessors_are_named():
    src = sources()
    everything = "\n".join(src.values())
    hip = "\n".join(t for f, t in src.items() if f.endswith(".hip"))
    names = set(re.findall(r"__global__[^;{]*?\b(k_\w+)\s*\(", hip))
    names |= set(re.findall(r"__device__[^;{=]*?\b(\w+)\s*\([^;{]*\)\s*(?:const\s*)?\{", hip)) - {"operator"}
    names |= set(re.findall(r"^struct (\w+)", hip, flags=re.M))
    assert len(names) > 80
    unused = sorted(n for n in names if len(re.findall(r"\b%s\b" % re.escape(n), everything)) < 2)
    assert not unused, unused
