"""Builds the HIP library (libidf.so) for gfx950 with hipcc, and the way into it from Python (push.cpp), in-tree."""
from __future__ import annotations

import glob
import os
import shlex
import subprocess
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libidf.so")
PUSH_SRC = os.path.join(CSRC, "push.cpp")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def extra_flags():
    """Further hipcc flags from the environment (IDF_HIPCC_FLAGS), e.g. -D switches of a timing build."""
    return shlex.split(os.environ.get("IDF_HIPCC_FLAGS", ""))


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def push_path():
    """The extension module of this interpreter and this torch: it is tied to the binary interfaces of both, and another one's is another file."""
    import torch
    return os.path.join(HERE, f"_push.torch-{torch.__version__}{sysconfig.get_config_var('EXT_SUFFIX')}")


def push_command(out):
    """The extension module is host code against torch's own headers and libraries, which are in the process before it is loaded."""
    import torch
    from torch.utils.cpp_extension import include_paths, library_paths
    return ([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-o", out, PUSH_SRC,
             f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}"] +
            [a for d in [sysconfig.get_paths()["include"]] + include_paths() for a in ("-isystem", d)] +
            ["-L" + d for d in library_paths()] + ["-ltorch_python", "-ltorch_cpu", "-lc10"])


def up_to_date() -> bool:
    push = push_path()
    if not os.path.exists(LIB) or not os.path.exists(push) or os.path.getmtime(push) < os.path.getmtime(PUSH_SRC):
        return False
    deps = sources() + glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(ROOT, "include", "*.h"))
    return all(os.path.getmtime(LIB) >= os.path.getmtime(d) for d in deps)


def _run(cmd, verbose=False):
    # the host pass does not know the GPU-only feature switch and says so once per use: harmless
    noise = "is not a recognized feature for this target"
    if verbose:
        print(" ".join(cmd))
    proc = subprocess.run(cmd, stderr=subprocess.PIPE, text=True)
    err = "\n".join(l for l in proc.stderr.splitlines() if noise not in l)
    if err.strip():
        print(err)
    if proc.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed with code {proc.returncode}: {' '.join(cmd[-3:])}")


def build_push(verbose: bool = False) -> str:
    """Compile push.cpp into push_path() (put there whole: another process may be about to load it)."""
    path = push_path()
    part = f"{path}.{os.getpid()}"
    try:
        _run(push_command(part), verbose)
        os.replace(part, path)
    finally:
        if os.path.exists(part):
            os.remove(part)
    return path


def build_library(verbose: bool = False) -> str:
    """Compile every kernel and the host side into paper_1804_10727_amd/libidf.so."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(HERE, "build")
    os.makedirs(objdir, exist_ok=True)
    # one translation unit per kernel file, compiled side by side, then linked
    objs = [os.path.join(objdir, os.path.basename(f)[:-4] + ".o") for f in sources()]
    with ThreadPoolExecutor(max_workers=min(8, len(objs))) as ex:
        list(ex.map(lambda fo: _run([hipcc] + HIPCC_FLAGS + extra_flags() + ["-c", "-o", fo[1], fo[0]], verbose), zip(sources(), objs)))
    _run([hipcc, "--offload-arch=gfx950", "-fPIC", "-shared", "-o", LIB] + objs, verbose)
    return LIB


def build(force: bool = True, verbose: bool = False) -> str:
    """Both of them; returns the library's path."""
    if not force and up_to_date():
        return LIB
    with ThreadPoolExecutor(max_workers=1) as ex:
        push = ex.submit(build_push, verbose)
        build_library(verbose)
        push.result()
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
