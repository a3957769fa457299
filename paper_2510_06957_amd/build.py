"""Build libtstgemm.so (HIP, gfx950 only) in-tree with hipcc, and _launch, the binding's native half (host code on torch's C++
headers), with g++.  The second needs the headers of Python and torch; where it cannot be built, the binding does without.

    python -m paper_2510_06957_amd.build

Packed-fp32 instruction selection is switched off for the device code
(-Xclang -target-feature -Xclang -packed-fp32-ops); the host pass warns that it does not
know the feature, which is harmless.
"""
from __future__ import annotations

import os
import pathlib
import shutil
import subprocess
import sys
import sysconfig

HERE = pathlib.Path(__file__).resolve().parent
ROOT = HERE.parent
CSRC = HERE / "csrc"
LIB = HERE / "libtstgemm.so"
LAUNCH = HERE / ("_launch" + sysconfig.get_config_var("EXT_SUFFIX"))   # of this Python; the torch it is for is in the module
SOURCES = ["tcsc_host.cpp", "reblock.hip", "tstgemm_side.hip", "tstgemm_large.hip", "tstgemm_small.hip", "tstgemm_matrix.hip",
           "tstgemm_decode.hip", "tstgemm_packed.hip", "probes.hip", "tstgemm_noalloc.hip"]
ARCH = "gfx950"


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found: libtstgemm needs the ROCm toolchain")
    return exe


def command(out: pathlib.Path = LIB, extra: list[str] | None = None) -> list[str]:
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-shared", "-x", "hip",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-Wall", "-Wno-unused-command-line-argument",
           f"-I{ROOT / 'include'}", f"-I{CSRC}"]
    cmd += [str(CSRC / s) for s in SOURCES]
    cmd += extra or []
    cmd += ["-o", str(out)]
    return cmd


def launch_command(out: pathlib.Path = LAUNCH) -> list[str]:
    import torch
    home = pathlib.Path(torch.__file__).resolve().parent
    cmd = [shutil.which("g++") or "g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall",
           "-DUSE_ROCM", "-D__HIP_PLATFORM_AMD__=1", f'-DBUILT_FOR_TORCH="{torch.__version__}"', f"-I{ROOT / 'include'}", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"]
    for path in (home / "include", home / "include" / "torch" / "csrc" / "api" / "include",
                 pathlib.Path(hipcc()).resolve().parent.parent / "include", sysconfig.get_paths()["include"]):
        cmd += ["-isystem", str(path)]
    cmd += [str(CSRC / "launch.cpp"), f"-L{home / 'lib'}", "-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10", "-o", str(out)]
    return cmd


def _run(cmd: list[str], verbose: bool):
    if verbose:
        print(" ".join(cmd))
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
    if r.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed ({r.returncode}):\n{err}")
    if verbose and err.strip():
        print(err)


def build(verbose: bool = False) -> pathlib.Path:
    _run(command(), verbose)
    try:
        _run(launch_command(), verbose)
    except (RuntimeError, ImportError, OSError) as e:   # no g++, no headers, no torch
        LAUNCH.unlink(missing_ok=True)
        print(f"{LAUNCH.name} was not built (calls from Python take 3 us longer without it): {e}", file=sys.stderr)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
