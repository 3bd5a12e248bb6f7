"""Build libbsr_actprune.so (HIP, gfx950) and the extension module over it, in-tree.

``python -m paper_2311_16883_amd.build`` compiles every ``csrc/*.hip`` file for
gfx950 and links them into ``paper_2311_16883_amd/libbsr_actprune.so`` (hipcc
cross-compiles without a GPU), then compiles ``csrc/torch_calls.cpp`` into
``paper_2311_16883_amd/_torch_calls_<torch version>.<ABI tag>.so`` (see
``calls_path``), which calls that library with torch tensors as arguments.
"""
from __future__ import annotations

import os
import re
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor
from pathlib import Path

PKG = Path(__file__).resolve().parent
ROOT = PKG.parent
CSRC = PKG / "csrc"
OBJ = PKG / "_build"
LIB = PKG / "libbsr_actprune.so"

HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
ROCM_INCLUDE = Path(HIPCC).resolve().parent.parent / "include"

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option",
    "-Wno-unused-function",
    f"-I{ROOT / 'include'}", f"-I{CSRC}",
]



def calls_path() -> Path:
    """The extension module.  It fits one interpreter ABI and one build of torch, and its name says which: a module
    left by another of either is not found and a new one is built, where loading it could crash."""
    import torch
    return PKG / f"_torch_calls_{re.sub('[^0-9A-Za-z]+', '_', torch.__version__)}{sysconfig.get_config_var('EXT_SUFFIX')}"


def sources():
    return sorted(CSRC.glob("*.hip"))


def build_library(verbose: bool = False, jobs: int = 8) -> Path:
    OBJ.mkdir(exist_ok=True)

    def compile_one(src: Path) -> Path:
        obj = OBJ / (src.stem + ".o")
        cmd = [HIPCC, *FLAGS, "-c", str(src), "-o", str(obj)]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        # the host pass does not know the packed-fp32 target feature; that warning is expected
        # (and the global -> LDS copies of dw_wide.hip set M0 inside inline assembly, which the
        # backend remarks on once per call site)
        err = "\n".join(l for l in r.stderr.splitlines()
                        if "packed-fp32-ops" not in l and "reserved registers: m0" not in l
                        and "Reserved registers on the clobber list" not in l)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src.name}:\n{r.stderr}")
        if verbose and err.strip():
            print(err, flush=True)
        return obj

    with ThreadPoolExecutor(max_workers=min(jobs, 16)) as ex:
        objs = list(ex.map(compile_one, sources()))
    tmp = LIB.with_suffix(f".{os.getpid()}.tmp")
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-fno-gpu-rdc", "-o", str(tmp), *map(str, objs)]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, LIB)
    build_calls(verbose)
    return LIB


def build_calls(verbose: bool = False) -> Path:
    """The extension module: host code only, needs the library to link against."""
    import torch
    from torch.utils.cpp_extension import include_paths, library_paths
    path = calls_path()
    tmp = path.with_suffix(f".{os.getpid()}.tmp")
    rocm = ROCM_INCLUDE if ROCM_INCLUDE.exists() else Path("/opt/rocm/include")
    cmd = [HIPCC, "-x", "c++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f"-I{ROOT / 'include'}",
           *(f"-isystem{p}" for p in [*include_paths(), sysconfig.get_paths()["include"], str(rocm)]),
           str(CSRC / "torch_calls.cpp"), "-x", "none", "-o", str(tmp), f"-L{PKG}", "-lbsr_actprune", "-Wl,-rpath,$ORIGIN",
           *(f"-L{p}" for p in library_paths()), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on torch_calls.cpp:\n{r.stderr}")
    os.replace(tmp, path)
    return path


if __name__ == "__main__":
    print(build_library(verbose="-v" in sys.argv))
