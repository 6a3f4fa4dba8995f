"""Build the HIP libraries in-tree for gfx950: ``paper_2604_18002_amd/libngc.so`` (the method) and
``paper_2604_18002_amd/libngc_probe.so`` (streaming probes for the measurement harness); with the host compiler
``paper_2604_18002_amd/_ngc_host.so`` (the Python front of the C ABI) and, where torch is there to compile against,
``paper_2604_18002_amd/libngc_torch.so`` (its reader of torch tensors)."""
from __future__ import annotations

import os
import shutil
import subprocess
import sysconfig

_PKG = os.path.dirname(os.path.abspath(__file__))
_CSRC = os.path.join(_PKG, "csrc")
LIB_PATH = os.path.join(_PKG, "libngc.so")
PROBE_LIB_PATH = os.path.join(_PKG, "libngc_probe.so")   # measurement probes, not part of the method
HOST_LIB_PATH = os.path.join(_PKG, "_ngc_host.so")       # CPython front of the C ABI (no device code)
TORCH_LIB_PATH = os.path.join(_PKG, "libngc_torch.so")   # the front's reader of torch tensors (no device code)

_COMMON = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
           # packed fp32 instructions stay off on the test machines
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]

# (source, extra flags).  The eviction units hold the exactly specified noise
# arithmetic: no contraction there.
_UNITS = (
    ("ngc_evict.hip", ["-ffp-contract=off"]),
    ("ngc_paged.hip", ["-ffp-contract=off"]),
    ("ngc_attn.hip", []),
    ("ngc_score.hip", []),
    ("ngc_replay.hip", []),
)
_PROBE_UNITS = (("ngc_probe.hip", []),)


def _hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found; the HIP library cannot be built")
    return exe


def torch_identity(torch) -> str:
    """Names the torch that the reader of tensors is compiled against; it serves no other."""
    return f"{torch.__version__} {getattr(torch.version, 'git_version', None)}"


def build(verbose: bool = False) -> str:
    """Compile every translation unit and link the shared library.  Always
    recompiles (this is the 'does it build' check)."""
    hipcc = _hipcc()
    bdir = os.path.join(_PKG, "_build")
    os.makedirs(bdir, exist_ok=True)
    for units, lib in ((_UNITS, LIB_PATH), (_PROBE_UNITS, PROBE_LIB_PATH)):
        objs = []
        for src, extra in units:
            obj = os.path.join(bdir, src.replace(".hip", ".o"))
            cmd = [hipcc, *_COMMON, *extra, "-c", os.path.join(_CSRC, src), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            r = subprocess.run(cmd, capture_output=True, text=True)
            if r.returncode != 0:
                raise RuntimeError(f"hipcc failed on {src}:\n{r.stderr}")
            objs.append(obj)
        cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", lib, *objs]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"link failed:\n{r.stderr}")
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        raise RuntimeError("no host C++ compiler found; the Python front cannot be built")
    python = ["-I", sysconfig.get_paths()["include"]]
    cmd = [cxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall"]
    host_units = [("ngc_host.cpp", HOST_LIB_PATH, ["-ldl"])]
    try:
        import torch
    except ImportError:      # the front needs none: without the reader it asks the tensors' methods
        torch = None
    if torch is not None:
        from torch.utils.cpp_extension import include_paths, library_paths
        host_units.append(("ngc_torch.cpp", TORCH_LIB_PATH, [
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DNGC_TORCH_IDENTITY="{torch_identity(torch)}"',
            *(f"-isystem{d}" for d in include_paths()), *(f"-L{d}" for d in library_paths()),
            "-ltorch_python", "-ltorch_cpu", "-lc10"]))
    for src, lib, flags in host_units:
        r = subprocess.run([*cmd, *python, os.path.join(_CSRC, src), "-o", lib, *flags], capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"{cxx} failed on {src}:\n{r.stderr}")
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose=True))
