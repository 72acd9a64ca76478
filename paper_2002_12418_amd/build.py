"""Builds libmnnconv.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree.

    python -m paper_2002_12418_amd.build
"""
from __future__ import annotations

import hashlib
import importlib.util
import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(os.path.dirname(PKG), "include")
OBJ_DIR = os.path.join(PKG, "_build")
LIB_PATH = os.path.join(PKG, "libmnnconv.so")

SOURCES = ["api.cpp", "transforms.hip", "transforms_rect.hip", "transforms_short.hip", "products_short.hip", "gemm.hip", "gemm_split.hip", "gemm_short.hip", "conv_patch.hip", "conv_short.hip", "gemm_prepared.hip", "weight_layout.hip", "fill.hip", "static_scratch.hip", "wino_fused.hip", "wino_full.hip", "wino_cols.hip", "gemm_bf16.hip", "strassen.hip", "microbench.hip"]

# -packed-fp32-ops is switched off: hand-checked scalar fp32 code only.
COMMON = ["-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950", "-I", INCLUDE, "-I", CSRC,
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument",
          "-Wno-unknown-warning-option"]


def _hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: the HIP library cannot be built")


def _compile(src: str) -> str:
    obj = os.path.join(OBJ_DIR, os.path.splitext(src)[0] + ".o")
    extra = os.environ.get("MNNCONV_EXTRA_HIPCC_FLAGS", "").split()      # e.g. -DNAME=value for tuning experiments
    cmd = [_hipcc(), "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj] + COMMON + extra
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
    warn = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip())
    if warn:
        sys.stderr.write(warn + "\n")
    return obj


def _torch_dir():
    spec = importlib.util.find_spec("torch")
    return spec.submodule_search_locations[0] if spec else None


def fast_call_path():
    """The file of the short way from Python into the library (fast_call.cpp), None without torch or the source.  It reads torch's tensors where the
    headers it was compiled against have their members, so the name says for which torch, Python, source and C interface it is."""
    torch_dir = _torch_dir()
    if torch_dir is None:
        return None
    h = hashlib.sha256(sys.version.encode())
    try:
        for f in (os.path.join(torch_dir, "version.py"), os.path.join(CSRC, "fast_call.cpp"), os.path.join(INCLUDE, "mnn_conv.h")):
            with open(f, "rb") as fp:
                h.update(fp.read())
    except OSError:
        return None
    return os.path.join(PKG, f"_fast_call_{h.hexdigest()[:16]}.so")


def fast_call_command(out: str, *flags: str) -> list:
    """Compiles fast_call.cpp against the headers of the torch that is installed."""
    torch_dir = _torch_dir()
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", *flags, "-I", INCLUDE,
            "-I", sysconfig.get_paths()["include"], "-I", os.path.join(torch_dir, "include"), "-I", "/opt/rocm/include",
            os.path.join(CSRC, "fast_call.cpp"), "-o", out, "-L", os.path.join(torch_dir, "lib"),
            "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]


def build_fast_call() -> None:
    path = fast_call_path()
    if path is None:
        raise RuntimeError("torch not found")
    tmp = f"{path}.{os.getpid()}.tmp"
    r = subprocess.run(fast_call_command(tmp), capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed on fast_call.cpp:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, path)
    for f in os.listdir(PKG):                              # of other sources or versions
        if f.startswith("_fast_call") and f.endswith(".so") and f != os.path.basename(path):
            os.remove(os.path.join(PKG, f))


def build_library(verbose: bool = True) -> str:
    """Compile every source for gfx950 and link paper_2002_12418_amd/libmnnconv.so."""
    os.makedirs(OBJ_DIR, exist_ok=True)
    wanted = {os.path.splitext(src)[0] + ".o" for src in SOURCES}
    for stale in os.listdir(OBJ_DIR):                      # objects of sources that were renamed or removed
        if stale.endswith(".o") and stale not in wanted:
            os.remove(os.path.join(OBJ_DIR, stale))
    with ThreadPoolExecutor(max_workers=min(6, len(SOURCES))) as ex:
        fast = ex.submit(build_fast_call)
        objs = list(ex.map(_compile, SOURCES))
        try:
            fast.result()
        except (RuntimeError, OSError) as e:               # the library and the binding's general path need neither torch nor g++
            sys.stderr.write(f"the short call path is not built: {e}\n")
    tmp = LIB_PATH + ".tmp"
    cmd = [_hipcc(), "-shared", "-fPIC", "--offload-arch=gfx950", "-o", tmp] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB_PATH)
    if verbose:
        print(f"built {LIB_PATH} ({os.path.getsize(LIB_PATH) // 1024} KiB)")
    return LIB_PATH


if __name__ == "__main__":
    build_library()
