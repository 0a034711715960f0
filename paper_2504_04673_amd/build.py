"""Build step: compiles the HIP sources in csrc/ into libsagnn.so for gfx950 (in-tree)."""
from __future__ import annotations

import os
import subprocess
import sysconfig
import warnings
from concurrent.futures import ThreadPoolExecutor

_HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(_HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(_HERE), "include")
LIB = os.path.join(_HERE, "libsagnn.so")
# csrc/marshal.c, the calls of binding.py: for one interpreter's headers, which its name carries
MARSHAL_SOURCE = os.path.join(CSRC, "marshal.c")
MARSHAL = os.path.join(_HERE, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))
OBJDIR = os.path.join(_HERE, "_build")
SOURCES = ["api.hip", "pack.hip", "plan.hip", "spmm.hip", "spmm_flat.hip", "spmm_sweep.hip", "gemm_nn_bf16.hip", "gemm_nn_fp32.hip", "gemm_nn_bf16x3.hip", "gemm.hip", "stages.hip", "radix.hip",
           "fused.hip", "permute.hip", "sweep_plan.hip", "tiles.hip"]
HEADERS = [os.path.join(CSRC, "common.h"), os.path.join(CSRC, "rowload.h"), os.path.join(CSRC, "gemm.h"),
           os.path.join(CSRC, "gemm_nn.h"), os.path.join(INCLUDE, "sagnn.h")]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
    # packed fp32 VALU ops are kept off (plain v_fma_f32 only)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-pass-failed",
]


def sources():
    return [os.path.join(CSRC, s) for s in SOURCES if os.path.exists(os.path.join(CSRC, s))]


def stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    return any(os.path.getmtime(d) > t for d in sources() + HEADERS) or marshal_stale()


def marshal_stale() -> bool:
    return not os.path.exists(MARSHAL) or os.path.getmtime(MARSHAL_SOURCE) > os.path.getmtime(MARSHAL)


def _run(cmd, verbose):
    res = subprocess.run(cmd, capture_output=True, text=True)
    if verbose or res.returncode != 0:
        print(res.stdout)
        print(res.stderr)
    if res.returncode != 0:
        raise RuntimeError("compilation failed: " + " ".join(cmd[-3:]))


def build_hip(verbose: bool = False, incremental: bool = False, jobs: int = 8) -> str:
    """Compile every source to an object file (in parallel) and link libsagnn.so.  With
    incremental=True only sources newer than their object file are recompiled."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJDIR, exist_ok=True)
    hdr_t = max(os.path.getmtime(h) for h in HEADERS)
    todo, objs = [], []
    for src in sources():
        obj = os.path.join(OBJDIR, os.path.basename(src) + ".o")
        objs.append(obj)
        fresh = (incremental and os.path.exists(obj)
                 and os.path.getmtime(obj) > max(os.path.getmtime(src), hdr_t))
        if not fresh:
            todo.append([hipcc, *HIPCC_FLAGS, f"-I{INCLUDE}", "-c", "-o", obj, src])
    with ThreadPoolExecutor(max_workers=max(1, jobs)) as ex:
        list(ex.map(lambda c: _run(c, verbose), todo))
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs], verbose)
    try:
        build_marshal(verbose)
    except (OSError, RuntimeError) as e:      # no C compiler, headers or x86-64: binding.py has ctypes then
        if os.path.exists(MARSHAL):
            os.remove(MARSHAL)                # (of another source)
        warnings.warn(f"calls go through ctypes: {e}")
    return LIB


def build_marshal(verbose: bool = False) -> str:
    """Compiled beside its place and moved there whole: another process may be loading it."""
    part = f"{MARSHAL}.{os.getpid()}"
    try:
        _run([os.environ.get("CC", "gcc"), "-O2", "-Wall", "-shared", "-fPIC", "-I" + sysconfig.get_paths()["include"], "-o", part,
              MARSHAL_SOURCE], verbose)
        os.replace(part, MARSHAL)
    finally:
        if os.path.exists(part):
            os.remove(part)
    return MARSHAL
