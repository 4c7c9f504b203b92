"""Build libakvq.so (hand-written HIP for gfx950) in-tree with hipcc, and the Python side of its decode calls with g++."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libakvq.so")
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


def build_nowait(out: str) -> str:
    """The library again, behind build(), with a pivot scoring that looks for other workgroups' statistics only once (a test of
    what a workgroup does that does not find them)."""
    obj = os.path.join(CSRC, "akvq_select_nowait.o")
    subprocess.run([HIPCC, *FLAGS, "-DAKVQ_ONCE_POLLS=0", "-c", os.path.join(CSRC, "akvq_select.hip"), "-o", obj], check=True,
                   stderr=subprocess.DEVNULL)
    objs = [os.path.join(CSRC, src.replace(".hip", ".o")) for src in SOURCES if src != "akvq_select.hip"]
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", out, *objs, obj], check=True)
    return out


def build(verbose: bool = False) -> str:
    """Compile every kernel source and link the shared library.  Always recompiles."""
    objs = []
    procs = []
    for src in SOURCES:
        obj = os.path.join(CSRC, src.replace(".hip", ".o"))
        cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{out}")
        if verbose and out.strip():
            print(out)
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    subprocess.run(cmd, check=True)
    build_native()
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
