"""Build the C-ABI library (attention forward, bf16 GEMM, FP8 MoE) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
import warnings
from concurrent.futures import ThreadPoolExecutor

_HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(_HERE, "csrc")
OBJ_DIR = os.path.join(_HERE, "_build")
LIB_PATH = os.path.join(_HERE, "libattn_mi355x.so")
NATIVE_SRC = "native_calls.cpp"                      # the Python binding's plain calls, against torch's C++ interface
NATIVE_PATH = os.path.join(_HERE, "_native" + sysconfig.get_config_var("EXT_SUFFIX"))     # (for this Python only)
SOURCES = ["attn_api.cpp", "attn_fwd_kernel.hip", "attn_split_kernel.hip", "gemm_api.cpp", "gemm_bf16_kernel.hip",
           "gemm_unaligned_kernel.hip", "moe_api.cpp", "moe_fp8_kernel.hip"]
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed-fp32 instructions are kept out of all device code: some of their forms have given wrong results on this hardware
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def hipcc_path() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    return "hipcc"


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass does not know the device-only target feature and says so: harmless
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if verbose and out.strip():
        print(out, flush=True)


def _newest_header() -> float:
    dirs = (CSRC, os.path.join(os.path.dirname(_HERE), "include"))
    return max(os.path.getmtime(os.path.join(d, f)) for d in dirs for f in os.listdir(d) if f.endswith(".h"))


def stale_sources() -> list:
    """Sources and headers that are newer than the built library (empty if there is none to compare with)."""
    if not os.path.exists(LIB_PATH):
        return []
    t = os.path.getmtime(LIB_PATH)
    dirs = (CSRC, os.path.join(os.path.dirname(_HERE), "include"))
    return sorted(f for d in dirs for f in os.listdir(d) if f != NATIVE_SRC and os.path.getmtime(os.path.join(d, f)) > t)


def _native_command(out):
    """One command compiles and links the extension module; torch's libraries are the ones the process has loaded."""
    import torch
    from torch.utils.cpp_extension import include_paths
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    includes = [*include_paths(), sysconfig.get_paths()["include"]]
    return [hipcc_path(), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wno-unused-command-line-argument", "-DUSE_ROCM", '-DNATIVE_TORCH="%s"' % torch.__version__,
            "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), *("-isystem" + p for p in includes),
            "-o", out, os.path.join(CSRC, NATIVE_SRC), "-L" + lib, "-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10"]


def build_library(verbose: bool = False, incremental: bool = False) -> str:
    """Compile every source of the library under csrc/ (one hipcc per file, in parallel), link libattn_mi355x.so, then
    build the extension module, which C programs do without.  Always recompiles unless `incremental`, which keeps the
    objects that are newer than their source and than every header."""
    os.makedirs(OBJ_DIR, exist_ok=True)
    hipcc, hdr = hipcc_path(), _newest_header()
    objs, jobs = [], []
    for s in SOURCES:
        src, obj = os.path.join(CSRC, s), os.path.join(OBJ_DIR, s + ".o")
        objs.append(obj)
        if incremental and os.path.exists(obj) and os.path.getmtime(obj) > max(os.path.getmtime(src), hdr):
            continue
        jobs.append([hipcc, *HIPCC_FLAGS, "-c", "-o", obj, src])
    with ThreadPoolExecutor(max(1, min(len(jobs), os.cpu_count() or 1))) as ex:
        list(ex.map(lambda c: _run(c, verbose), jobs))
    tmp = LIB_PATH + ".tmp.%d" % os.getpid()
    try:
        _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs], verbose)
    except RuntimeError:
        if os.path.exists(tmp):
            os.remove(tmp)
        raise
    os.replace(tmp, LIB_PATH)
    try:
        build_native(verbose, incremental)
    except (ImportError, RuntimeError) as why:           # (without torch, or without its headers: a C program needs neither)
        warnings.warn("the extension module was not built, Python calls take longer: %s" % why)
    return LIB_PATH


def build_native(verbose: bool = False, incremental: bool = False) -> None:
    """Compile and link the extension module, which is optional: without it the binding's calls take the longer way."""
    src, record = os.path.join(CSRC, NATIVE_SRC), os.path.join(OBJ_DIR, NATIVE_SRC + ".command")
    tmp = NATIVE_PATH + ".tmp.%d" % os.getpid()
    try:
        command = "\n".join(_native_command(NATIVE_PATH))           # (torch's version and Python's folders among its words)
        if incremental and os.path.exists(NATIVE_PATH) and os.path.exists(record) and os.path.getmtime(NATIVE_PATH) > max(os.path.getmtime(src), _newest_header()):
            with open(record) as f:
                if f.read() == command:
                    return
        _run([tmp if word == NATIVE_PATH else word for word in command.split("\n")], verbose)
        os.replace(tmp, NATIVE_PATH)
        with open(record, "w") as f:
            f.write(command)
    except (ImportError, RuntimeError):
        if os.path.exists(NATIVE_PATH):
            os.remove(NATIVE_PATH)                       # (made for an older library, or another torch)
        raise
    finally:
        if os.path.exists(tmp):
            os.remove(tmp)


if __name__ == "__main__":
    print(build_library(verbose=True, incremental="--incremental" in sys.argv))
