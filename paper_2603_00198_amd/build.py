"""Build libstrd.so (HIP kernels + C ABI) for gfx950 with hipcc and strd_host.so (the binding's native half) with g++, in-tree."""
from __future__ import annotations

import glob
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libstrd.so")
HOST = os.path.join(PKG, "strd_host.so")   # the binding's native half, a Python extension module

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# A change of flags or toolchain has to keep two properties of the generated code, both checked by
# tests/test_host_logic.py from the compiler's resource report: the kernels that split LDS reads into
# issue and wait (ssd_mfma.hip, ssd_seg_mfma.hip, attn_mfma.hip) must fit their register budget with
# no scratch, no spilled VGPR / SGPR and no accumulation registers -- a register moved between the two
# halves of a split read would carry stale data; and matrix products must take their operands from
# ordinary VGPRs (-amdgpu-mfma-vgpr-form), which those budgets assume.
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument", "-mllvm", "-amdgpu-mfma-vgpr-form", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
]


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, os.path.basename(src) + ".o")
    cmd = [HIPCC] + FLAGS + ["-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, err))
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _host_flags():
    import sysconfig

    import torch
    from torch.utils import cpp_extension
    inc = cpp_extension.include_paths("cuda") + [sysconfig.get_paths()["include"], os.path.join(ROOT, "include")]
    tlib = os.path.join(os.path.dirname(torch.__file__), "lib")
    cxx = ["-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-DUSE_ROCM=1", "-w",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI)] + ["-I" + i for i in inc]
    # torch's own libraries are in the process before the module is; libstrd.so lies beside it
    link = ["-L" + tlib, "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_hip", "-ltorch_python", "-L" + PKG, "-l:libstrd.so",
            "-Wl,-rpath,$ORIGIN"]
    return cxx, link


def _compile_host() -> str:
    obj = os.path.join(OBJ, "host.cpp.o")
    subprocess.check_call(["g++"] + _host_flags()[0] + ["-c", os.path.join(CSRC, "host.cpp"), "-o", obj])
    return obj


def build(verbose: bool = True) -> str:
    """Compile every csrc/*.hip and link the shared library, then the binding's host module; always rebuilds."""
    os.makedirs(OBJ, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    with ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        host = ex.submit(_compile_host)
        objs = list(ex.map(_compile, srcs))
        host_obj = host.result()
    tmp = LIB + ".tmp.%d" % os.getpid()
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs +
                          ["-L/opt/rocm/lib", "-lrocblas"])   # rocBLAS: the plain projection products of the block glue
    os.replace(tmp, LIB)
    tmp = HOST + ".tmp.%d" % os.getpid()
    subprocess.check_call(["g++", "-shared", "-o", tmp, host_obj] + _host_flags()[1])
    os.replace(tmp, HOST)
    if verbose:
        print("built", LIB, "from", len(srcs), "sources")
    return LIB


if __name__ == "__main__":
    build()
