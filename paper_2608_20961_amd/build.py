"""Build libtreewy.so from csrc/ with hipcc for gfx950, and the Python binding's native call path (_binding.so, host
code only) against the installed torch (both in-tree).

    python -m paper_2608_20961_amd.build
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
from typing import Optional

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
OBJDIR = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libtreewy.so")
BINDING = os.path.join(PKG, "_binding.so")
SOURCES = ["api.hip", "verify.hip", "small.hip", "prefill.hip", "commit.hip", "snapshot.hip", "tree.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
         # no packed-fp32 instructions anywhere in the device code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", INCLUDE, "-I", CSRC]


def binding_command(obj: str) -> Optional[list]:
    """g++ over binding.cpp (no device code) with torch's and HIP's headers; None where torch is not installed."""
    import sysconfig

    try:
        import torch
        from torch.utils import cpp_extension
    except ImportError:
        return None
    rocm = os.path.dirname(os.path.dirname(shutil.which(HIPCC) or "/opt/rocm/bin/hipcc"))
    inc = [*cpp_extension.include_paths(), sysconfig.get_paths()["include"], os.path.join(rocm, "include")]
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-Wall", "-DUSE_ROCM=1", "-D__HIP_PLATFORM_AMD__=1",
            "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), *[x for i in inc for x in ("-isystem", i)],
            "-I", INCLUDE, "-c", os.path.join(CSRC, "binding.cpp"), "-o", obj]


def link_binding(obj: str) -> None:
    """Links the binding; torch's libraries and libtreewy.so are in the process when it is imported."""
    from torch.utils import cpp_extension
    tmp = BINDING + ".tmp%d" % os.getpid()
    libs = [x for d in cpp_extension.library_paths() for x in ("-L", d, "-Wl,-rpath-link," + d)]
    subprocess.run(["g++", "-shared", "-fPIC", "-o", tmp, obj, "-L", PKG, "-Wl,-rpath,$ORIGIN", "-l:libtreewy.so", *libs,
                    "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip"], check=True)
    os.replace(tmp, BINDING)


def build(verbose: bool = False) -> str:
    """Both libraries; where torch is not installed the C-ABI library alone."""
    os.makedirs(OBJDIR, exist_ok=True)
    objs = [os.path.join(OBJDIR, src.replace(".hip", ".o")) for src in SOURCES]
    commands = {src: [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj] for src, obj in zip(SOURCES, objs)}
    binding_obj = os.path.join(OBJDIR, "binding.o")
    binding = binding_command(binding_obj)
    if binding:
        commands["binding.cpp"] = binding
    procs = {}
    for src, cmd in commands.items():
        if verbose:
            print(" ".join(cmd), flush=True)
        procs[src] = subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    failed = []
    for src, p in procs.items():
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if out.strip() and (verbose or p.returncode):
            print(out, file=sys.stderr)
        if p.returncode:
            failed.append(src)
    if set(failed) <= {"binding.cpp"}:                   # (the library does not depend on the binding)
        tmp = LIB + ".tmp%d" % os.getpid()
        subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs], check=True)
        os.replace(tmp, LIB)
    if failed:
        raise RuntimeError("the compiler failed on " + ", ".join(failed))
    if binding:
        link_binding(binding_obj)
    else:
        print("torch is not installed: built %s without the Python binding's native call path" % LIB, file=sys.stderr)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
