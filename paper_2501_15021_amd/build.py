"""Build libakvq.so (hand-written HIP for gfx950) in-tree with hipcc, and the Python side of its decode calls with g++."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libakvq.so")
NOWAIT = os.path.join(HERE, "libakvq_nowait.so")
SOURCES = ["akvq_api.hip", "akvq_quantize.hip", "akvq_decode.hip", "akvq_select.hip", "akvq_fold.hip", "akvq_stream.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-mllvm", "-amdgpu-mfma-vgpr-form",   # keep MFMA accumulators in VGPRs: no AGPR<->VGPR copies around VALU use
         "-Wall", "-Wno-unused-function"]
NATIVE = os.path.join(HERE, "_akvq_torch.so")


def build_native() -> str:
    """Compile _akvq_torch.so (host code only) against libakvq.so and the installed torch."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension

    lib_dir = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           *[f"-isystem{p}" for p in cpp_extension.include_paths()], "-isystem/opt/rocm/include",
           "-I" + sysconfig.get_paths()["include"], "-Wall", os.path.join(CSRC, "akvq_torch.cpp"), "-o", NATIVE,
           "-L" + lib_dir, "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip",
           "-L" + HERE, "-l:" + os.path.basename(LIB), "-Wl,-rpath,$ORIGIN"]
    subprocess.run(cmd, check=True)
    return NATIVE


def build(verbose: bool = False) -> str:
    """Compile every kernel source and link the shared library, and with it NOWAIT: the same library with a pivot scoring that looks for
    other workgroups' statistics only once (a test of what a workgroup does that does not find them).  Always recompiles."""
    jobs = [(src, src.replace(".hip", ".o"), []) for src in SOURCES] + [("akvq_select.hip", "akvq_select_nowait.o", ["-DAKVQ_ONCE_POLLS=0"])]
    for lib in (LIB, NOWAIT):  # none of an earlier build stays where this one fails
        if os.path.exists(lib):
            os.remove(lib)
    procs = []
    for src, obj, extra in jobs:
        cmd = [HIPCC, *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", os.path.join(CSRC, obj)]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((obj, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    failed = []
    for obj, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            failed.append(f"hipcc failed on {obj}:\n{out}")
        elif verbose and out.strip():
            print(out)
    if failed:
        raise RuntimeError("\n".join(failed))
    objs = [os.path.join(CSRC, src.replace(".hip", ".o")) for src in SOURCES]
    select, nowait = (os.path.join(CSRC, obj) for obj in ("akvq_select.o", "akvq_select_nowait.o"))
    for lib, parts in ((LIB, objs), (NOWAIT, [nowait if obj == select else obj for obj in objs])):
        subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", lib, *parts], check=True)
    build_native()
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
