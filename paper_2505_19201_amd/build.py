"""Builds libdream.so (the C-ABI HIP library) for gfx950 with hipcc.

`python -m paper_2505_19201_amd.build` compiles every csrc/*.hip to an object in csrc/_build/
(in parallel) and links them into paper_2505_19201_amd/libdream.so; csrc/call.cpp becomes the extension
paper_2505_19201_amd/_call.so through which the binding calls it.
"""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libdream.so")
CALL = os.path.join(HERE, "_call.so")
ARCH = "gfx950"

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}", "-I" + INCLUDE, "-I" + CSRC,
    "-Wall", "-Wno-unused-function", "-Wno-unknown-warning-option",
    # keep the compiler from forming packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # the first 14 dwords of a kernel's plain arguments in scalar registers when a wave starts: the arguments of a launch are in no cache, and reading
    # them is a trip to memory ahead of everything else
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    return "hipcc"


def _run(cmd):
    p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in p.stdout.splitlines() if "packed-fp32-ops" not in l)
    if p.returncode != 0:
        raise RuntimeError("command failed: %s\n%s" % (" ".join(cmd), out))
    return out


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _call_command(out: str):
    """Host compiler only: the extension holds no GPU code and finds libdream.so beside itself."""
    from torch.utils import cpp_extension
    import torch
    inc = ["-I" + d for d in (sysconfig.get_paths()["include"], INCLUDE, *cpp_extension.include_paths())]
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-w", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *inc,
            os.path.join(CSRC, "call.cpp"), "-o", out, "-L" + HERE, "-l:libdream.so", "-Wl,-rpath,$ORIGIN", "-L" + lib, "-ltorch_python", "-ltorch_cpu", "-lc10"]


def is_stale() -> bool:
    if not (os.path.exists(LIB) and os.path.exists(CALL)):
        return True
    t = min(os.path.getmtime(LIB), os.path.getmtime(CALL))
    deps = sources() + [os.path.join(CSRC, "call.cpp")] + glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(INCLUDE, "*.h"))
    return any(os.path.getmtime(d) > t for d in deps)


def build(verbose: bool = True, extra_flags=()) -> str:
    """Compile everything (always recompiles) and return the path of libdream.so."""
    bdir = os.path.join(CSRC, "_build")
    os.makedirs(bdir, exist_ok=True)
    hipcc = _hipcc()
    objs = []
    jobs = []
    for src in sources():
        obj = os.path.join(bdir, os.path.basename(src)[:-4] + ".o")
        objs.append(obj)
        jobs.append([hipcc, *HIPCC_FLAGS, *extra_flags, "-c", src, "-o", obj])
    with ThreadPoolExecutor(max_workers=min(8, len(jobs))) as ex:
        for out in ex.map(_run, jobs):
            if verbose and out.strip():
                print(out)
    tmp = LIB + ".tmp.%d" % os.getpid()
    out = _run([hipcc, "-shared", "-fPIC", f"--offload-arch={ARCH}", "-o", tmp, *objs])
    if verbose and out.strip():
        print(out)
    os.replace(tmp, LIB)
    tmp = CALL + ".tmp.%d" % os.getpid()
    _run(_call_command(tmp))
    os.replace(tmp, CALL)
    return LIB


if __name__ == "__main__":
    print(build(extra_flags=sys.argv[1:]))
