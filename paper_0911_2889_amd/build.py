"""Build the HIP library libflamefront.so for gfx950 (in-tree).

Every translation unit is compiled by hipcc for --offload-arch=gfx950 with
packed-FP32 instructions disabled, then linked into one shared library next
to this file. Run ``python -m paper_0911_2889_amd.build``.
"""

import concurrent.futures
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
OUT = os.path.join(HERE, "libflamefront.so")
BUILD_DIR = os.path.join(ROOT, "_build")
SOURCES = ["flame_kernels.hip", "mixed_kernels.hip", "resident_kernel.hip", "physical_kernels.hip",
           "ensemble_kernel.hip", "adjoint_kernels.hip", "circle_kernels.hip", "flame_api.hip"]
ARCH = "gfx950"


def hipcc():
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: the HIP toolchain is required to build libflamefront.so")


def common_flags():
    return [
        "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
        "-I", CSRC, "-I", INCLUDE, "-Wall", "-Wno-unused-function",
    ]


def _compile(src, verbose, extra, build_dir):
    obj = os.path.join(build_dir, os.path.splitext(src)[0] + ".o")
    cmd = [hipcc()] + common_flags() + list(extra) + ["-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{res.stdout}\n{res.stderr}")
    return obj


def build(verbose=False, extra_flags=(), out=OUT):
    """Compile and link; extra_flags (e.g. tuning macros) go to every hipcc compile."""
    build_dir = BUILD_DIR if out == OUT else os.path.join(BUILD_DIR, os.path.basename(out) + ".d")
    os.makedirs(build_dir, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose, extra_flags, build_dir), SOURCES))
    tmp = out + ".tmp"
    cmd = [hipcc(), "-shared", f"--offload-arch={ARCH}", "-fPIC"] + objs + ["-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link failed:\n{res.stdout}\n{res.stderr}")
    os.replace(tmp, out)
    return out


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
