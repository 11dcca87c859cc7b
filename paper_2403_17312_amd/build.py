"""Builds the HIP library (libswa_hip.so) for gfx950, in-tree, with hipcc."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import warnings
from concurrent.futures import ThreadPoolExecutor
from typing import Optional

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB_PATH = os.path.join(HERE, "libswa_hip.so")
NATIVE_PATH = os.path.join(HERE, "_swa_native.so")
SOURCES = ["swa_api.hip", "swa_decode.hip", "swa_short.hip", "swa_short_shared.hip", "swa_compact.hip", "swa_prefill.hip", "swa_quant.hip", "swa_flash.hip", "swa_offload.hip", "swa_splitk.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
    "-Wall", "-Wno-unused-command-line-argument",
]


# MFMA kernels: keep the accumulators in ordinary vector registers (no copies in and out of the
# accumulation file around every softmax step).
EXTRA = {f: ["-mllvm", "-amdgpu-mfma-vgpr-form=1"] for f in ("swa_flash.hip", "swa_prefill.hip")}


def _compile(src: str) -> str:
    obj = os.path.join(CSRC, src.replace(".hip", ".o"))
    cmd = [HIPCC] + FLAGS + EXTRA.get(src, []) + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build_native() -> Optional[str]:
    """Compile the binding's native half (an extension module that reads torch tensors; host code only).  Without a host compiler or
    the headers of torch and Python there is none, and the binding does without."""
    import sysconfig

    import torch
    root = os.path.dirname(torch.__file__)
    needs = [os.path.join(root, "include", "torch", "csrc", "autograd", "python_variable.h"),
             os.path.join(sysconfig.get_paths()["include"], "Python.h")]
    missing = [f for f in needs if not os.path.exists(f)] + ([] if shutil.which("g++") else ["g++"])
    if missing:
        if os.path.exists(NATIVE_PATH):
            os.remove(NATIVE_PATH)                       # (of another build: its calls may not be this library's)
        warnings.warn(f"the binding's native half is not built, for want of {', '.join(missing)}: calls convert their arguments in Python")
        return None
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DSWA_TORCH_VERSION="{torch.__version__}"',
           "-I", os.path.join(ROOT, "include"), "-isystem", os.path.join(root, "include"),
           "-isystem", os.path.join(root, "include", "torch", "csrc", "api", "include"), "-isystem", "/opt/rocm/include",
           "-isystem", sysconfig.get_paths()["include"], os.path.join(CSRC, "swa_native.cpp"), "-o", NATIVE_PATH,
           "-L", os.path.join(root, "lib"), "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10_hip", "-lc10"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed on swa_native.cpp:\n{r.stderr}")
    return NATIVE_PATH


def build(verbose: bool = False) -> str:
    """Compile every HIP source, link libswa_hip.so, and compile the binding's native half.  Always recompiles."""
    with ThreadPoolExecutor(max_workers=4) as ex:
        native = ex.submit(build_native)
        objs = list(ex.map(_compile, SOURCES))
        native.result()
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB_PATH] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    if verbose:
        print("built", LIB_PATH)
    return LIB_PATH


if __name__ == "__main__":
    build(verbose=True)
