"""Build the HIP library libdftpicard.so in-tree for gfx950.

Usage: python -m paper_0910_1531_amd.build  (or paper_0910_1531_amd.build.build()).
Every call recompiles.  Objects and the device assembly hipcc keeps for
inspection go to paper_0910_1531_amd/_build/.
"""
import concurrent.futures
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libdftpicard.so")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")

SOURCES = ["dft_host.cpp", "ct_launch_z1_f32.hip", "ct_launch_y_f32.hip", "ct_launch_y_f64.hip", "ct_launch_z1_f64.hip",
           "ct_launch_zwide_f32.hip", "ct_launch_zwide_f64.hip", "ct_launch_z1_more_f32.hip", "ct_launch_z1_more_f64.hip", "ct_launch_x2_f64.hip", "ct_launch_x2_alt_f64.hip",
           "ct_launch_z2.hip", "ct_launch_x2_f32.hip", "ct_launch_x2_alt_f32.hip", "ct_launch_x.hip", "dft_kernels.hip",
           "ct_launch_screen.hip", "dft_tune.hip", "dft_adjoint.hip", "dft_screen.hip", "dft_api.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function", "-I", CSRC, "-I", INCLUDE]
DEVICE = ["--offload-arch=" + ARCH, "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-munsafe-fp-atomics", "-ffp-contract=on"]


def _compile(src):
    path = os.path.join(CSRC, src)
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    if src.endswith(".hip"):
        cmd = [HIPCC, "-x", "hip"] + DEVICE + COMMON + ["-save-temps=obj", "-c", path, "-o", obj]
    else:
        cmd = [HIPCC, "-x", "c++"] + COMMON + ["-c", path, "-o", obj]
    r = subprocess.run(cmd, cwd=BUILD, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    return obj, r.stderr


def build(verbose=False):
    """Compile every source and link the shared library; returns its path."""
    os.makedirs(BUILD, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(len(SOURCES), os.cpu_count() or 8)) as ex:
        results = list(ex.map(_compile, SOURCES))
    objs = [o for o, _ in results]
    if verbose:
        for (o, err) in results:
            if err.strip():
                print(err, file=sys.stderr)
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=" + ARCH, "-shared", "-fPIC", "-o", tmp] + objs + ["-lamdhip64"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    shutil.move(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
