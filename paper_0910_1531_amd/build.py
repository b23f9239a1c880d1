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
           "ct_launch_zwide_f32.hip", "ct_launch_zwide_f64.hip", "ct_launch_z1_more_f32.hip", "ct_launch_z1_more_f64.hip",
           "ct_launch_z2.hip", "ct_launch_x.hip", "dft_kernels.hip", "ct_launch_screen.hip", "dft_tune.hip", "dft_adjoint.hip",
           "dft_screen.hip", "dft_api.hip"]
# The X2 kernels: one code object per precision, class (the Hessian product in FP64 only) and group of row lengths.
X2_CLASSES = {"double": range(4), "float": (0, 2)}
X2_GROUPS = 6


def units():
    """(object name, source, macro definitions) of every translation unit, the longest to compile first."""
    out = [(os.path.splitext(s)[0], s, []) for s in SOURCES]
    out += [(f"ct_launch_x2_{t}_{c}_{g}", "ct_launch_x2.hip", [f"-DDFT_X2_T={t}", f"-DDFT_X2_CLASS={c}", f"-DDFT_X2_GROUP={g}"])
            for t, classes in X2_CLASSES.items() for c in classes for g in range(X2_GROUPS)]
    return out


HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function", "-I", CSRC, "-I", INCLUDE]
DEVICE = ["--offload-arch=" + ARCH, "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-munsafe-fp-atomics", "-ffp-contract=on"]


def _compile(unit):
    name, src, defs = unit
    path = os.path.join(CSRC, src)
    cwd = os.path.join(BUILD, name)   # each unit's own folder: the files hipcc keeps are named after the source
    os.makedirs(cwd, exist_ok=True)
    obj = os.path.join(cwd, name + ".o")
    if src.endswith(".hip"):
        cmd = [HIPCC, "-x", "hip"] + DEVICE + COMMON + defs + ["-save-temps=obj", "-c", path, "-o", obj]
    else:
        cmd = [HIPCC, "-x", "c++"] + COMMON + ["-c", path, "-o", obj]
    r = subprocess.run(cmd, cwd=cwd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    return obj, r.stderr


def build(verbose=False):
    """Compile every source and link the shared library; returns its path."""
    os.makedirs(BUILD, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=os.cpu_count() or 8) as ex:
        results = list(ex.map(_compile, units()))
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
