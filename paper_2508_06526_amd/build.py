"""Build libpikv.so (gfx950 HIP kernels + C ABI) in-tree with hipcc, and with g++ the CPython extension
_pikv_native.so that binding.py makes its calls through.

    python -m paper_2508_06526_amd.build
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libpikv.so")
NATIVE = os.path.join(HERE, "_pikv_native.so")
SOURCES = ["pikv_api.hip", "pikv_route.hip", "pikv_attn.hip", "pikv_utility.hip", "pikv_evict.hip", "pikv_step.hip", "pikv_aux.hip",
           "pikv_policy.hip"]

# packed-fp32 instructions are switched off for all device code (the compiler would
# otherwise form v_pk_*_f32 from ordinary float math)
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)

    def compile_one(src):
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        cmd = [hipcc] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        out = "\n".join(l for l in r.stdout.splitlines()
                        if "packed-fp32-ops" not in l and "is not a recognized feature" not in l)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed for %s:\n%s" % (src, r.stdout))
        if verbose and out.strip():
            print(out)
        return obj

    def compile_native():
        """Against the headers of the torch it will be loaded beside (same C++ ABI), its libraries' symbols left to it."""
        import sysconfig
        import torch
        from torch.utils import cpp_extension
        tmp = NATIVE + ".tmp%d" % os.getpid()
        include = cpp_extension.include_paths() + [sysconfig.get_paths()["include"], "/opt/rocm/include", os.path.join(ROOT, "include")]
        cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-w", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
               "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI)] + ["-I" + d for d in include]
        libs = os.path.join(os.path.dirname(torch.__file__), "lib")
        cmd += [os.path.join(CSRC, "pikv_binding.cpp"), "-o", tmp, "-L" + libs, "-ltorch_python", "-ltorch", "-lc10", "-lc10_hip"]
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        if r.returncode != 0:
            raise RuntimeError("g++ failed for pikv_binding.cpp:\n%s" % r.stdout)
        os.replace(tmp, NATIVE)

    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES) + 1)) as ex:
        native = ex.submit(compile_native)
        objs = list(ex.map(compile_one, SOURCES))
        native.result()
    tmp = LIB + ".tmp%d" % os.getpid()
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
    sys.exit(0)
