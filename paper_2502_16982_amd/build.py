"""Builds the HIP library in-tree for gfx950 (cross-compiles without a GPU)."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG_DIR, "csrc")
OBJ_DIR = os.path.join(PKG_DIR, "_build")
LIB_NAME = "libmuon_hip.so"
LIB_PATH = os.path.join(PKG_DIR, LIB_NAME)
MARSHAL_PATH = os.path.join(PKG_DIR, "_adamw_marshal.so")
# the planner is plain C++ (it also builds with g++ alone, see tests/test_plan_sanitized.py); the rest is HIP
SOURCES = ("muon_api.hip", "muon_plan.cpp", "kernels_ew.hip", "kernels_gemm_bf16.hip", "kernels_gemm_pair.hip", "kernels_gemm_f32.hip",
           "kernels_adamw.hip", "probe_mfma.hip")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed-fp32 VALU forms are kept out of generated code: some have given wrong results on this hardware
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # kernel arguments arrive in scalar registers with the wave instead of through a load it would start with: 0.25 to 0.3 us
    # of each dependent launch (step of one 128 x 256 matrix in fp32 64.3 -> 59.3 us, nine small matrices 107.9 -> 103.6)
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Wno-unused-command-line-argument",
]


def hipcc_path() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: the Muon HIP library cannot be built")


def marshal_stamp() -> str:
    """What the extension is compiled for: it reads tensors through torch's inlined C++, whose layouts belong to one torch."""
    import torch
    return f"torch {torch.__version__} {torch.version.git_version} python {sys.version_info[0]}.{sys.version_info[1]}"


def marshal_command(out):
    """The compiler line of the extension that marshals AdamW's tensors (host code only; torch's headers and libraries)."""
    import sysconfig
    import torch
    from torch.utils import cpp_extension
    lib_dir = os.path.join(os.path.dirname(torch.__file__), "lib")
    include = [*cpp_extension.include_paths(), sysconfig.get_paths()["include"]]
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            f'-DMUON_BUILT_FOR="{marshal_stamp()}"',
            *(f"-isystem{d}" for d in include), os.path.join(CSRC, "adamw_marshal.cpp"), "-o", out, f"-L{PKG_DIR}",
            f"-l:{LIB_NAME}", f"-L{lib_dir}", "-ltorch_python", "-ltorch_cpu", "-lc10", "-Wl,-rpath,$ORIGIN"]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError(f"{os.path.basename(cmd[0])} failed:\n" + " ".join(cmd) + "\n" + proc.stdout + proc.stderr)


def build_marshal(verbose: bool = False) -> bool:
    """Builds the extension that marshals AdamW's tensors.  It is optional: where torch, its headers, Python's or g++ are
    missing the library is complete without it and the binding reads the tensors in Python (False, the reason on stderr)."""
    tmp = MARSHAL_PATH + ".tmp"
    try:
        _run(marshal_command(tmp), verbose)
    except (ImportError, AttributeError, OSError, RuntimeError) as e:
        if os.path.exists(tmp):
            os.remove(tmp)
        print(f"{os.path.basename(MARSHAL_PATH)} was not built, muon_adamw_step reads its tensors in Python: "
              f"{type(e).__name__}: {e}", file=sys.stderr, flush=True)
        return False
    os.replace(tmp, MARSHAL_PATH)
    return True


def build_library(verbose: bool = False, extra_flags=()) -> str:
    """Compiles every source (in parallel, one object each) and links the shared library, with hipcc alone; then the optional
    extension.  Always recompiles."""
    hipcc = hipcc_path()
    os.makedirs(OBJ_DIR, exist_ok=True)
    objs = [os.path.join(OBJ_DIR, os.path.splitext(s)[0] + ".o") for s in SOURCES]
    cmds = [[hipcc, *HIPCC_FLAGS, *extra_flags, "-c", os.path.join(CSRC, s), "-o", o] for s, o in zip(SOURCES, objs)]
    with ThreadPoolExecutor(max_workers=min(8, len(cmds))) as pool:
        list(pool.map(lambda c: _run(c, verbose), cmds))
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB_PATH + ".tmp"], verbose)
    if os.path.exists(MARSHAL_PATH):             # of another library, maybe of another torch: never beside this one
        os.remove(MARSHAL_PATH)
    os.replace(LIB_PATH + ".tmp", LIB_PATH)
    build_marshal(verbose)
    return LIB_PATH


if __name__ == "__main__":
    print(build_library(verbose=True))
