"""Build liblsb.so (all HIP sources, gfx950) and the Python layer's native
marshalling module ``_bind.so`` in-tree with hipcc.

Usage: ``python -m paper_0912_0947_amd.build`` or ``build()`` from Python.
Both land next to this file.
"""
from __future__ import annotations

import glob
import os
import shutil
import subprocess
import sys
import time

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblsb.so")
BIND = os.path.join(HERE, "_bind.so")
BIND_SOURCE = os.path.join(CSRC, "bind", "lsb_bind.cpp")
ARCH = os.environ.get("LSB_OFFLOAD_ARCH", "gfx950")

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
    "--offload-arch=" + ARCH,
    # no packed fp32 instructions anywhere in the library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"),
]


ROCM_LIB = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "lib")
# roctx ranges around the serving loop's phases (rocprofv3 --marker-trace)
LINK_FLAGS = ["-L" + ROCM_LIB, "-lrocprofiler-sdk-roctx", "-Wl,-rpath," + ROCM_LIB]


def sources() -> list[str]:
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.cpp")))


def _hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: the HIP library cannot be built")


def bind_command(out: str) -> list[str]:
    """Command that builds the marshalling module against this Python and
    its torch (host code only)."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension

    dirs = [sysconfig.get_paths()["include"], *cpp_extension.include_paths(), os.path.join(ROOT, "include")]
    libs = os.path.join(os.path.dirname(torch.__file__), "lib")
    return [_hipcc(), "-x", "c++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1",
            "-DUSE_ROCM=1", "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
            *[x for d in dirs for x in ("-isystem", d)], "-isystem", os.path.join(os.path.dirname(ROCM_LIB), "include"),
            BIND_SOURCE, "-o", out, "-L" + libs, "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip",
            "-Wl,-rpath," + libs]


def start_bind(out: str) -> subprocess.Popen | None:
    """Start the marshalling module's build; None if this torch cannot say how."""
    try:
        return subprocess.Popen(bind_command(out), stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    except (ImportError, OSError, RuntimeError) as e:
        print("the marshalling module cannot be built: %s" % e, file=sys.stderr, flush=True)
        return None


def finish_bind(proc: subprocess.Popen | None, out: str) -> bool:
    """Put the built marshalling module in place.  Without it every call still
    works, through the checked path, so its failure does not fail the build;
    a module of an earlier build must not stay beside the new library."""
    text = proc.communicate()[0] if proc else ""
    if proc and proc.returncode == 0:
        os.replace(out, BIND)
        return True
    print("the marshalling module was not built; calls will take the checked path\n" + text, file=sys.stderr, flush=True)
    if os.path.exists(BIND):
        os.remove(BIND)
    return False


def build(verbose: bool = False, jobs: int = 8) -> str:
    """Compile every source to an object (in parallel), then link liblsb.so;
    the marshalling module builds beside them."""
    hipcc = _hipcc()
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    t0 = time.time()
    bind_tmp = BIND + ".tmp%d" % os.getpid()
    bind = start_bind(bind_tmp)
    procs = []
    objs = []
    for src in sources():
        obj = os.path.join(objdir, os.path.basename(src) + ".o")
        objs.append(obj)
        cmd = [hipcc, *HIPCC_FLAGS, "-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        while sum(p.poll() is None for _, p in procs) >= jobs:
            time.sleep(0.05)
    failed = []
    for src, p in procs:
        out, _ = p.communicate()
        if p.returncode != 0:
            failed.append((src, out))
        elif out.strip() and verbose:
            print(out)
    if failed:
        msg = "\n".join("%s:\n%s" % (s, o) for s, o in failed)
        raise RuntimeError("hipcc failed:\n" + msg)
    tmp = LIB + ".tmp%d" % os.getpid()
    subprocess.check_call([hipcc, "-shared", "-fPIC", "--offload-arch=" + ARCH, "-o", tmp, *objs, *LINK_FLAGS])
    os.replace(tmp, LIB)
    finish_bind(bind, bind_tmp)
    if verbose:
        print("built %s in %.1f s" % (LIB, time.time() - t0), flush=True)
    return LIB


if __name__ == "__main__":
    build(verbose="-q" not in sys.argv)
