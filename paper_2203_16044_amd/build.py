"""Build libqs.so (HIP, gfx950) in-tree: one object per source, compiled in parallel, then linked."""
from __future__ import annotations

import concurrent.futures as cf
import glob
import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(ROOT, "_build", "obj")
LIB = os.path.join(PKG, "libqs.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
CFLAGS = [
    "-O3", "-std=c++17", f"--offload-arch={ARCH}", "-fPIC", "-fvisibility=hidden",
    # packed FP32 instructions stay off: plain float code only
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]

# The kernels that interpret op tables branch on scalars. Left as branches (not rewritten into if-then-else regions) their
# cases update a thread's amplitudes in place: tiles 101 instead of 154 registers, four tiles a CU; complex64 block
# passes of 12 qubits without spills. A 40-circuit complex64 batch 660 -> 557 us, SU(4) layers on 31 qubits 297 -> 291
# ms, their complex64 form on 27 qubits 19.3 -> 18.7 ms.
FILE_FLAGS = {f: ["-mllvm", "-structurizecfg-skip-uniform-regions=1"] for f in ("qs_tile.hip", "qs_block.hip", "qs_small.hip")}


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.cpp")))


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, os.path.basename(src) + ".o")
    cmd = [HIPCC, *CFLAGS, *FILE_FLAGS.get(os.path.basename(src), []), "-c", src, "-o", obj]
    if src.endswith(".cpp"):
        cmd[1:1] = ["-x", "hip"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip())
    if err:
        print(err, file=sys.stderr)
    return obj


def build(jobs: int | None = None) -> str:
    os.makedirs(OBJ, exist_ok=True)
    srcs = sources()
    jobs = jobs or min(len(srcs), int(os.environ.get("MAX_JOBS", os.cpu_count() or 4)), 16)
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    return LIB


SANITIZE_DIR = os.path.join(ROOT, "_build", "sanitize")
# host code only: AddressSanitizer + UndefinedBehaviorSanitizer on the CPU side (planner, validation, ABI); the GPU
# code objects are built as usual
SANITIZE_FLAGS = ["-Xarch_host", "-fsanitize=address,undefined", "-Xarch_host", "-fno-sanitize-recover=undefined",
                  "-Xarch_host", "-fno-omit-frame-pointer", "-Xarch_host", "-g"]


def build_sanitized(jobs: int | None = None) -> str:
    """libqs with sanitized host code, in _build/sanitize (selected at run time with QS_LIBQS)."""
    global OBJ, LIB, CFLAGS
    saved = OBJ, LIB, CFLAGS
    OBJ, LIB = os.path.join(SANITIZE_DIR, "obj"), os.path.join(SANITIZE_DIR, "libqs.so")
    CFLAGS = CFLAGS + SANITIZE_FLAGS
    try:
        os.makedirs(OBJ, exist_ok=True)
        srcs = sources()
        jobs = jobs or min(len(srcs), int(os.environ.get("MAX_JOBS", os.cpu_count() or 4)), 16)
        with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
            objs = list(ex.map(_compile, srcs))
        tmp = LIB + ".tmp"
        cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-Xarch_host", "-fsanitize=address,undefined",
               "-shared-libsan", "-o", tmp, *objs]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"link failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
        os.replace(tmp, LIB)
        return LIB
    finally:
        OBJ, LIB, CFLAGS = saved


if __name__ == "__main__":
    print(build_sanitized() if "--sanitize" in sys.argv else build())
