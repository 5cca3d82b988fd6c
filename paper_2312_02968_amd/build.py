"""Build the HIP library libmondpm.so in-tree for gfx950.

    python -m paper_2312_02968_amd.build        (or build() from Python)

Each .hip file under csrc/ is compiled by hipcc to an object in _build/ and
the objects are linked into paper_2312_02968_amd/libmondpm.so, which the
Python binding loads.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
BUILD = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libmondpm.so")

ARCH = os.environ.get("MONDPM_ARCH", "gfx950")
HIPCC = os.environ.get("HIPCC", shutil.which("hipcc") or "/opt/rocm/bin/hipcc")

COMMON = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    # no packed FP32 instructions in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
    "-Wno-unused-result",
]


def _sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


# pm_fft.hip is compiled once per box size (and once for the rest, part 0):
# its instantiations take minutes in one translation unit
FFT_PARTS = (1024, 512, 256, 128, 64, 32, 16, 0)


def _jobs():
    jobs = []
    for src in _sources():
        if os.path.basename(src) == "pm_fft.hip":
            jobs = [(src, n) for n in FFT_PARTS] + jobs
        else:
            jobs.append((src, None))
    return jobs


def _compile(src, part=None, defines=(), build_dir=BUILD):
    tag = "" if part is None else f".{part}"
    obj = os.path.join(build_dir, os.path.basename(src) + tag + ".o")
    if part is not None:
        defines = (*defines, f"PM_FFT_PART={part}")
    cmd = [HIPCC, *COMMON, *[f"-D{d}" for d in defines], "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def build(verbose=False, defines=(), lib=LIB, build_dir=BUILD) -> str:
    """Compile and link; defines (NAME=VALUE) set compile-time launch shapes."""
    os.makedirs(build_dir, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=8) as ex:
        objs = list(ex.map(lambda j: _compile(j[0], j[1], defines, build_dir), _jobs()))
    tmp = lib + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, lib)
    if verbose:
        print("built", lib)
    return lib


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
