"""Compile the HIP sources under csrc/ for gfx950 into libbrgemm_gfx950.so (in-tree)."""
import glob
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libbrgemm_gfx950.so")
FASTCALL = os.path.join(HERE, "_fastcall" + sysconfig.get_config_var("EXT_SUFFIX"))     # for this Python alone

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-command-line-argument", "-Wno-inline-asm"]


def _compile(src):
    obj = os.path.join(OBJ, os.path.basename(src) + ".o")
    r = subprocess.run([HIPCC, *FLAGS, "-c", src, "-o", obj], capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build_fastcall(cc: str = "gcc"):
    """The binding's native way into the library (host only).  Without a C compiler or Python's headers there
    is none, and its calls go through ctypes."""
    for old in (FASTCALL, os.path.join(HERE, "_fastcall.so")):
        if os.path.exists(old):
            os.remove(old)
    try:
        subprocess.run([cc, "-O2", "-std=c11", "-Wall", "-shared", "-fPIC", "-I" + sysconfig.get_paths()["include"],
                        os.path.join(CSRC, "fastcall.c"), "-o", FASTCALL], check=True)
    except (OSError, subprocess.CalledProcessError) as e:
        sys.stderr.write(f"{os.path.basename(FASTCALL)} not built, calls go through ctypes: {e}\n")
        return None
    return FASTCALL


def build(jobs: int = 8) -> str:
    os.makedirs(OBJ, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(_compile, srcs))
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-fno-gpu-rdc", *objs, "-o", LIB], check=True)
    build_fastcall()
    return LIB


if __name__ == "__main__":
    print(build())
