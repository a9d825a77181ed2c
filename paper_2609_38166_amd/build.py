"""Build the HIP library libleapquant.so in-tree for gfx950.

hipcc cross-compiles without a GPU.  Flags: -O3, IEEE fp32 division and square
root (hipcc's default), denormals kept, packed-fp32 instructions disabled.
Each source is compiled to an object of its own (with the scheduler options of
SCHED below) and the objects are linked into the library.
"""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import tempfile
import warnings
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
LIB = os.path.join(PKG, "libleapquant.so")
# measurement helpers for bench.py (not part of the method's C ABI)
BENCH_LIB = os.path.join(PKG, "libleapquant_bench.so")
# argument marshalling of the Python binding (host code, against torch's headers)
MARSHAL_LIB = os.path.join(PKG, "_marshal.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CXX = "g++"

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-fno-gpu-flush-denormals-to-zero",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]

# Machine scheduler options per source file (the LLVM AMDGPU backend's), each
# measured against the default on the KDA workload (8192 tiles, W = 64, r = 8):
#  - decode: the max-ILP strategy, 1.7% less time per launch over the window
#    positions (2.2% on the GQA GDN layer), no spill;
#  - tile kernel: the AMDGPU register-pressure trackers, for the scalar gate's
#    exports, which spill without them: 8192 E4M3 states with 33 records 291 us
#    instead of 255 (2048: 76 and 73); commits and quantizations within 1%.
SCHED = {
    "lq_decode.hip": ["-mllvm", "-amdgpu-sched-strategy=max-ilp"],
    "lq_tile.hip": ["-mllvm", "-amdgpu-use-amdgpu-trackers"],
}


def sources():
    return sorted(glob.glob(os.path.join(PKG, "csrc", "*.hip")))


# A build-time alternative of the library, for measuring one design choice
# against its alternative (never loaded unless named in LEAPQUANT_LIB):
# the decode's integer code product on the vector ALU instead of the matrix cores.
VALU_CP_LIB = os.path.join(PKG, "libleapquant_valucp.so")


def _compile(srcs, out, verbose, defines=()):
    inc = ["-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc")]
    with tempfile.TemporaryDirectory() as td:
        def obj(src):
            o = os.path.join(td, os.path.basename(src) + ".o")
            cmd = [HIPCC, *FLAGS, *SCHED.get(os.path.basename(src), []), *defines, *inc, "-c", src, "-o", o]
            if verbose:
                print(" ".join(cmd), file=sys.stderr)
            subprocess.run(cmd, check=True)
            return o
        with ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
            objs = list(ex.map(obj, srcs))
        tmp = out + ".tmp"
        cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp]
        if verbose:
            print(" ".join(cmd), file=sys.stderr)
        subprocess.run(cmd, check=True)
    os.replace(tmp, out)


def _compile_marshal(verbose):
    """The extension saves the binding host time and is tied to this torch's headers;
    where it cannot be built, none is left and the binding does without it."""
    try:
        _build_marshal(verbose)
    except (ImportError, OSError, subprocess.CalledProcessError) as e:
        if os.path.exists(MARSHAL_LIB):
            os.remove(MARSHAL_LIB)
        warnings.warn(f"_marshal.so is not built, the binding will check calls in Python: {e}", RuntimeWarning)


def _build_marshal(verbose):
    import sysconfig

    import torch
    from torch.utils.cpp_extension import include_paths
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    inc = [os.path.join(ROOT, "include"), sysconfig.get_paths()["include"], "/opt/rocm/include", *include_paths()]
    tmp = MARSHAL_LIB + ".tmp"
    cmd = [CXX, "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-DUSE_ROCM", "-D__HIP_PLATFORM_AMD__",
           f'-DLQ_TORCH_VERSION="{torch.__version__}"',
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *(x for d in inc for x in ("-isystem", d)),
           os.path.join(PKG, "py_csrc", "marshal.cpp"), "-o", tmp,
           "-L", lib, "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    if verbose:
        print(" ".join(cmd), file=sys.stderr)
    subprocess.run(cmd, check=True)
    os.replace(tmp, MARSHAL_LIB)


def build(verbose: bool = False) -> str:
    with ThreadPoolExecutor(max_workers=1) as ex:
        marshal = ex.submit(_compile_marshal, verbose)
        _compile(sources(), LIB, verbose)
        marshal.result()
    _compile(sorted(glob.glob(os.path.join(PKG, "bench_csrc", "*.hip"))), BENCH_LIB, verbose)
    return LIB


def build_valu_code_product(verbose: bool = False) -> str:
    _compile(sources(), VALU_CP_LIB, verbose, defines=("-DLQ_CODE_PRODUCT_VALU",))
    return VALU_CP_LIB


if __name__ == "__main__":
    if "--valu-code-product" in sys.argv:
        print(build_valu_code_product(verbose=True))
    else:
        print(build(verbose=True))
