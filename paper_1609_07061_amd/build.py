"""Builds libqnn.so (hand-written HIP kernels for gfx950 behind the C ABI of include/qnn.h) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libqnn.so")
NATIVE = os.path.join(PKG, "_native.so")
NATIVE_STAMP = os.path.join(OBJ, "native.txt")  # what _native.so was built for
SOURCES = ["qnn_api.hip", "qnn_probe.hip", "qnn_pack.hip", "qnn_quant.hip", "qnn_dedup.hip", "qnn_conv_first.hip", "qnn_gemm_valu.hip", "qnn_gemm_slice.hip", "qnn_gemm_tile.hip", "qnn_gemm_mfma.hip", "qnn_gemm_mfma_k0.hip",
           "qnn_gemm_mfma_k1.hip", "qnn_gemm_mfma_k2.hip", "qnn_gemm_mfma_k3.hip", "qnn_gemm_mfma_k4.hip", "qnn_gemm_stage_k0.hip",
           "qnn_gemm_stage_k1.hip", "qnn_gemm_stage_k2.hip", "qnn_gemm_panel_k0.hip", "qnn_gemm_bytes_panel_k0.hip",
           "qnn_gemm_mixed.hip", "qnn_gemm_codes.hip", "qnn_gemm_image.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc", "-ffp-contract=off",
    # packed-fp32 instruction selection is switched off for every kernel of this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unknown-warning-option",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def _stale(target: str, deps: list[str]) -> bool:
    if not os.path.exists(target):
        return True
    t = os.path.getmtime(target)
    return any(os.path.getmtime(d) > t for d in deps)


def _deps(path: str, seen: set | None = None) -> list[str]:
    """The file and, recursively, the project headers it includes with #include "..."."""
    import re

    seen = set() if seen is None else seen
    if path in seen or not os.path.exists(path):
        return []
    seen.add(path)
    out = [path]
    for name in re.findall(r'^\s*#\s*include\s+"([^"]+)"', open(path).read(), flags=re.M):
        for d in (os.path.dirname(path), CSRC, os.path.join(ROOT, "include")):
            cand = os.path.join(d, name)
            if os.path.exists(cand):
                out += _deps(cand, seen)
                break
    return out


def build(force: bool = False, verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    jobs = []
    objs = []
    for src in SOURCES:
        s = os.path.join(CSRC, src)
        o = os.path.join(OBJ, src + ".o")
        objs.append(o)
        if force or _stale(o, _deps(s)):
            jobs.append([HIPCC, *FLAGS, "-c", s, "-o", o])

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"{cmd[0]} failed:\n" + " ".join(cmd) + "\n" + r.stdout + r.stderr)
        return r.stderr

    pool = ThreadPoolExecutor(max_workers=1)
    binding = pool.submit(_build_binding, run) if force or _binding_stale() else None
    with ThreadPoolExecutor(max_workers=min(8, max(1, len(jobs)))) as ex:
        for err in ex.map(run, jobs):
            if verbose and err.strip():
                print(err, file=sys.stderr)
    if force or jobs or _stale(LIB, objs):
        run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-fno-gpu-rdc", "-o", LIB, *objs])
    if binding is not None:
        binding.result()
    pool.shutdown()
    return LIB


def _built_for() -> str:
    """What the binding's native part depends on beside its source: this torch and this Python (as in __init__.py)."""
    import torch

    return f"torch {torch.__version__}, {sys.implementation.cache_tag}"


def _binding_stale() -> bool:
    if _stale(NATIVE, [os.path.join(CSRC, "qnn_binding.cpp")]) or not os.path.exists(NATIVE_STAMP):
        return True
    with open(NATIVE_STAMP) as f:
        return f.read() != _built_for()


def _build_binding(run) -> None:
    """The binding's native part, against the torch that is installed.  It only shortens the host side of some calls: where it cannot be
    built (no g++, no headers of torch or Python) the library is complete without it, and the package says so when it is imported."""
    import sysconfig

    import torch
    from torch.utils.cpp_extension import include_paths, library_paths

    src = os.path.join(CSRC, "qnn_binding.cpp")
    for old in (NATIVE, NATIVE_STAMP):
        if os.path.exists(old):
            os.remove(old)
    try:
        run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
             f'-DQNN_BUILT_FOR="{_built_for()}"', *[f"-I{d}" for d in (*include_paths(), sysconfig.get_paths()["include"])], src, "-o", NATIVE,
             *[f"-L{d}" for d in library_paths()], "-ltorch_python", "-ltorch_cpu", "-lc10"])
    except (OSError, RuntimeError) as e:
        print(f"the binding's native part was not built: {e}", file=sys.stderr)
        return
    with open(NATIVE_STAMP, "w") as f:
        f.write(_built_for())


if __name__ == "__main__":
    print(build(force="--force" in sys.argv, verbose=True))
