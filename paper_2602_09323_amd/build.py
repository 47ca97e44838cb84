"""Builds libcoopt_attn.so and the benchmark's libcoopt_probe.so (HIP, gfx950 only) in-tree with hipcc,
and the Python binding's native part with g++ and torch's headers.  The libraries need hipcc alone: where the
native part does not compile, that is said and the binding's ctypes path takes its calls.

    python -m paper_2602_09323_amd.build [--force]

hipcc cross-compiles without a GPU.  Objects go to ``_build/`` next to this file; the shared
library lands beside the Python binding so that it travels with the source tree.
"""
from __future__ import annotations

import concurrent.futures
import importlib.metadata
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libcoopt_attn.so")
PROBE_LIB = os.path.join(HERE, "libcoopt_probe.so")      # measurement aid, not the product
SOURCES = ["kv_write.hip", "decode.hip", "decode_flat.hip", "prefill.hip", "gather.hip"]
PROBE_SOURCES = ["probe.hip"]
BINDING = os.path.join(HERE, "_binding" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))
BINDING_SOURCE = "binding_native.cpp"                    # host code: tensors to pointers, no kernel
BINDING_STAMP = os.path.join(HERE, "_binding.built_for")   # the torch that it was last compiled against, or did not compile
HEADERS = [os.path.join(CSRC, h) for h in ("common.hpp", "attn_tile.hpp", "kv_quant.hpp",
                                          "decode_internal.hpp", "launch_grid.hpp", "prefill_deal.hpp")] + [
    os.path.join(ROOT, "include", "coopt_attn.h"), os.path.join(ROOT, "include", "coopt_probe.h")]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
         "-I" + os.path.join(ROOT, "include"),
         # packed-FP32 VALU forms are kept out of the generated code on purpose
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument"]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    return "hipcc"


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [_hipcc(), *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass does not know the device-only target feature; that warning is expected
    err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _torch_version() -> str:
    try:
        return importlib.metadata.version("torch")
    except importlib.metadata.PackageNotFoundError:
        return "none"


def _build_binding() -> None:
    import torch
    root = os.path.dirname(torch.__file__)
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           f'-DCOOPT_TORCH_VERSION="{torch.__version__}"',
           "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(root, "include"),
           "-I" + os.path.join(root, "include", "torch", "csrc", "api", "include"),
           "-I" + sysconfig.get_paths()["include"], os.path.join(CSRC, BINDING_SOURCE), "-o", BINDING,
           "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"g++ failed for {BINDING_SOURCE}:\n{res.stderr}")


def _try_binding() -> None:
    if os.path.exists(BINDING):
        os.remove(BINDING)                               # (one of older sources, if the compiler fails)
    try:
        _build_binding()
    except (RuntimeError, OSError, ImportError) as e:
        sys.stderr.write(f"the binding's native part was not built, ctypes takes its calls: {e}\n")
    with open(BINDING_STAMP, "w") as f:
        f.write(_torch_version())


def needs_build() -> bool:
    """Whether a source is newer than what was made of it, or torch is another than the native part was made for."""
    if not all(os.path.exists(p) for p in (LIB, PROBE_LIB, BINDING_STAMP)):
        return True
    newest = max(os.path.getmtime(p)
                 for p in [os.path.join(CSRC, s) for s in SOURCES + PROBE_SOURCES + [BINDING_SOURCE]] + HEADERS)
    if min(os.path.getmtime(p) for p in (LIB, PROBE_LIB, BINDING_STAMP)) < newest:
        return True
    with open(BINDING_STAMP) as f:
        return f.read() != _torch_version()


def build(force: bool = True) -> str:
    """Compile every HIP source for gfx950 and link the shared library.  Returns its path."""
    if not force and not needs_build():
        return LIB
    os.makedirs(BUILD, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=6) as pool:
        binding = pool.submit(_try_binding)
        objs = list(pool.map(_compile, SOURCES + PROBE_SOURCES))
        binding.result()
    for lib, n in ((LIB, objs[:len(SOURCES)]), (PROBE_LIB, objs[len(SOURCES):])):
        cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-fno-gpu-rdc", "-o", lib, *n]
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError("link failed:\n" + res.stderr)
    return LIB


if __name__ == "__main__":
    print(build(force=True))
