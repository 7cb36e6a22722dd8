"""Builds libcartridge.so (hand-written HIP for gfx950) in-tree with hipcc, and the binding's native half with g++.

`python -m paper_2506_06266_amd.build` compiles every csrc/*.hip to an object file and links
them, and csrc/pycall.cpp; they are rebuilt only when a source or header is newer unless force=True, the native half also
when another interpreter, PyTorch or command would build it.
"""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
ROOT = os.path.dirname(HERE)
LIB = os.environ.get("CART_LIB_OUT", os.path.join(HERE, "libcartridge.so"))
PYCALL = os.path.join(os.path.dirname(os.path.abspath(LIB)), "_pycall.so")
OBJ_DIR = os.environ.get("CART_OBJ_DIR", os.path.join(HERE, "_build"))

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option",
    "-I", os.path.join(ROOT, "include"),
] + os.environ.get("CART_EXTRA_FLAGS", "").split()


def _newest_header() -> float:
    hs = glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(ROOT, "include", "*.h"))
    return max(os.path.getmtime(h) for h in hs)


def _compile(src: str, force: bool) -> str:
    obj = os.path.join(OBJ_DIR, os.path.basename(src)[:-4] + ".o")
    if (not force and os.path.exists(obj)
            and os.path.getmtime(obj) > max(os.path.getmtime(src), _newest_header())):
        return obj
    cmd = [HIPCC, *FLAGS, "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s\n%s" % (src, r.stdout, r.stderr))
    noise = "is not a recognized feature"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _compile_pycall(force: bool) -> str:
    """csrc/pycall.cpp against the installed PyTorch (paths only: nothing of it is initialised here)."""
    import torch
    src = os.path.join(CSRC, "pycall.cpp")
    at = os.path.dirname(os.path.abspath(torch.__file__))
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wextra",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           "-isystem", os.path.join(at, "include"), "-isystem", os.path.join(at, "include", "torch", "csrc", "api", "include"),
           "-isystem", sysconfig.get_paths()["include"], "-I", os.path.join(ROOT, "include"), src, "-o", PYCALL,
           "-L", os.path.join(at, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    # what the module's ABI hangs on, beside the objects: the module is loaded whatever it was built for
    stamp, built_for = os.path.join(OBJ_DIR, "_pycall.stamp"), " ".join([torch.__version__, sysconfig.get_config_var("SOABI") or "", *cmd])
    if (not force and os.path.exists(PYCALL) and os.path.exists(stamp) and open(stamp).read() == built_for
            and os.path.getmtime(PYCALL) > max(os.path.getmtime(src), _newest_header())):
        return PYCALL
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed for %s:\n%s\n%s" % (src, r.stdout, r.stderr))
    if r.stderr.strip():
        sys.stderr.write(r.stderr)
    with open(stamp, "w") as f:
        f.write(built_for)
    return PYCALL


def build(force: bool = True, jobs: int = 8) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        pycall = ex.submit(_compile_pycall, force)
        objs = list(ex.map(lambda s: _compile(s, force), srcs))
        pycall.result()
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-fno-gpu-rdc", "-o", LIB, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n%s\n%s" % (r.stdout, r.stderr))
    return LIB


if __name__ == "__main__":
    print(build(force="--incremental" not in sys.argv))
