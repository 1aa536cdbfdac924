"""Builds `liblsq.so` (the C-ABI library of include/lsq.h) for gfx950 with hipcc, and `_calls.<interpreter>.so` (how Python calls it) with g++.

    python -m paper_2110_05722_amd.build

hipcc cross-compiles without a GPU.  Each translation unit is compiled on its
own (in parallel) and the objects are linked into one shared library that sits
next to this file, so it travels with the source tree.
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblsq.so")
OBJ_DIR = os.path.join(HERE, "_build", "liblsq.so")
SOURCES = ["api", "calibrate", "adam", "bias_dropout_residual", "bias_act_dropout", "heads", "embedding", "pad", "layernorm", "softmax",
           "ls_xent"]
# the interpreter's tag in the name: another Python does not find it (and the torch it was built with is checked when it is loaded)
CALLS = os.path.join(HERE, "_calls" + sysconfig.get_config_var("EXT_SUFFIX"))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CXX = os.environ.get("CXX", "g++")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-command-line-argument",
    # packed fp32 VALU forms are switched off for the device pass (the host pass warns that it
    # does not know the feature; that is harmless)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def _compile(name: str, obj_dir: str = OBJ_DIR, extra: tuple = ()) -> str:
    src = os.path.join(CSRC, name + ".hip")
    obj = os.path.join(obj_dir, name + ".o")
    r = subprocess.run([HIPCC, *FLAGS, *extra, "-c", src, "-o", obj], capture_output=True, text=True)
    noise = ("packed-fp32-ops", "1 warning generated")
    err = "\n".join(l for l in r.stderr.splitlines() if not any(n in l for n in noise))
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {name}.hip:\n{r.stderr}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build(verbose: bool = True, lib: str = LIB, obj_dir: str = OBJ_DIR, extra: tuple = ()) -> str:
    os.makedirs(obj_dir, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(lambda n: _compile(n, obj_dir, extra), SOURCES))
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", lib, *objs], check=True,
                   capture_output=not verbose)
    if verbose:
        print(f"built {lib}")
    if lib == LIB:
        build_calls(verbose)
    return lib


def build_calls(verbose: bool = True) -> str:
    """The CPython extension of csrc/calls.cpp (host code; linked against liblsq.so beside it and torch's libraries,
    which the process has loaded by then)."""
    import torch

    t = os.path.dirname(torch.__file__)
    inc = [os.path.join(t, "include"), os.path.join(t, "include", "torch", "csrc", "api", "include"), sysconfig.get_paths()["include"]]
    cmd = [CXX, "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           f'-DLSQ_TORCH_VERSION="{torch.__version__}"',
           *(f"-I{i}" for i in inc), os.path.join(CSRC, "calls.cpp"), "-o", CALLS, f"-L{HERE}", "-l:liblsq.so",
           f"-L{os.path.join(t, 'lib')}", "-ltorch_python", "-ltorch_cpu", "-lc10", "-Wl,-rpath,$ORIGIN"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"{CXX} failed on calls.cpp:\n{r.stderr}")
    untagged = os.path.join(HERE, "_calls.so")          # a build of before the tag: any Python would take it
    if os.path.exists(untagged):
        os.remove(untagged)
    if verbose:
        print(f"built {CALLS}")
    return CALLS


if __name__ == "__main__":
    build()
