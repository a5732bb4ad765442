"""Compile libflashd.so for gfx950 with hipcc (cross-compiles without a GPU) and the Python binding's
native part with g++."""
from __future__ import annotations

import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libflashd.so")
SOURCES = ("flashd_api.hip", "flashd_perkey.hip", "flashd_tile.hip", "flashd_tile_f32.hip", "flashd_wide.hip", "flashd_short.hip", "flashd_tile64.hip",
           "flashd_decode.hip", "flashd_decode16.hip", "flashd_stats.hip", "flashd_widen.hip")
HEADERS = ("flashd_common.h", "flashd_kernels.h", "flashd_mma.h", "flashd_plan.h", "flashd_rows.h", "flashd_tile_parts.h", "flashd_wide_regs.h", os.path.join("..", "..", "include", "flashd.h"))

FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-command-line-argument"]


BINDING = os.path.join(HERE, "_flashd_binding.so")
BINDING_SOURCE = os.path.join(CSRC, "flashd_binding.cpp")


def stale() -> bool:
    if not os.path.exists(LIB) or not os.path.exists(BINDING):
        return True
    t = min(os.path.getmtime(LIB), os.path.getmtime(BINDING))
    deps = [os.path.join(CSRC, s) for s in SOURCES + HEADERS] + [BINDING_SOURCE]
    return any(os.path.getmtime(d) > t for d in deps)


def build_binding(verbose: bool = False) -> str:
    import sysconfig

    import torch
    from torch.utils.cpp_extension import include_paths
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}",
           f'-DFLASHD_TORCH="{torch.__version__}"',
           *[a for d in (*include_paths(), sysconfig.get_paths()["include"]) for a in ("-isystem", d)],
           BINDING_SOURCE, "-o", BINDING, "-L", lib, "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10",
           f"-Wl,-rpath,{lib}"]
    if verbose:
        print(" ".join(cmd))
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed:\n" + r.stderr)
    return BINDING


def build(force: bool = True, verbose: bool = False) -> str:
    if not force and not stale():
        return LIB
    cmd = ["hipcc", *FLAGS, "-o", LIB, *[os.path.join(CSRC, s) for s in SOURCES]]
    if verbose:
        print(" ".join(cmd))
    r = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass does not know the packed-fp32 target feature and says so; drop that noise
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + err)
    if verbose and err.strip():
        print(err)
    build_binding(verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
