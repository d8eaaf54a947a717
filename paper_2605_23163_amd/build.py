"""Build libfdd.so for gfx950 with hipcc (cross-compiles without a GPU).

    python -m paper_2605_23163_amd.build [--asm]

Objects go to ``_build/`` at the repository root, the library next to this
file so that it travels with the source tree.
"""
from __future__ import annotations

import importlib.util
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libfdd.so")
# (named for this interpreter: another one does not load it)
MARSHAL = os.path.join(PKG, "_marshal" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-I" + os.path.join(ROOT, "include"),
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument"]
# The bf16 attention and vocabulary kernels produce no NaN from finite inputs (masked
# scores are -inf and every inf - inf is avoided by construction), so max/min need no NaN
# quieting there.  The fp32 attention kernel passes the caller's NaN and infinities on.
EXTRA = {"attn_bf16.hip": ["-fno-honor-nans", "-mno-amdgpu-ieee"],
         "unmask.hip": ["-fno-honor-nans", "-mno-amdgpu-ieee"]}


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


def _run(cmd):
    p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in p.stdout.splitlines() if "packed-fp32-ops" not in l)
    if p.returncode:
        raise RuntimeError("command failed: " + " ".join(cmd) + "\n" + out)
    if out.strip():
        print(out)


def marshal_command(out):
    """The compiler call for the binding's native argument marshalling, or None where torch, its headers or Python's are
    missing.  torch is looked up, not imported."""
    try:
        spec = importlib.util.find_spec("torch")
    except (ImportError, ValueError):
        spec = None
    python = sysconfig.get_paths()["include"]
    if spec is None or not spec.origin or not os.path.exists(os.path.join(python, "Python.h")):
        return None
    torch = os.path.dirname(spec.origin)
    if not os.path.isdir(os.path.join(torch, "include")):
        return None
    lib = os.path.join(torch, "lib")
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-I" + os.path.join(ROOT, "include"), "-I" + python,
            "-I" + os.path.join(torch, "include"), "-I" + os.path.join(torch, "include", "torch", "csrc", "api", "include"),
            os.path.join(CSRC, "marshal.cpp"), "-o", out, "-L" + lib, "-lc10", "-ltorch_cpu", "-ltorch_python"]


def build_marshal():
    """Builds the marshalling module, which the library does not need: without it the binding does the same in Python.
    Returns its path, or None if it could not be built; an older one does not stay."""
    old = [f for f in os.listdir(os.path.dirname(MARSHAL)) if f.startswith("_marshal.") and f.endswith(".so")]
    tmp = MARSHAL + f".{os.getpid()}.tmp"
    cmd = marshal_command(tmp)
    built = False
    if cmd:
        try:
            _run(cmd)
            built = True
        except (OSError, RuntimeError) as e:
            print(f"arguments will be marshalled in Python: {e}")
    for f in old:
        if not built or f != os.path.basename(MARSHAL):
            os.remove(os.path.join(os.path.dirname(MARSHAL), f))
    if not built:
        if os.path.exists(tmp):
            os.remove(tmp)
        return None
    os.replace(tmp, MARSHAL)
    return MARSHAL


def build(asm: bool = False, jobs: int = 4) -> str:
    bdir = os.path.join(ROOT, "_build")
    os.makedirs(bdir, exist_ok=True)
    objs = []
    cmds = []
    for src in sources():
        obj = os.path.join(bdir, os.path.basename(src)[:-4] + ".o")
        objs.append(obj)
        cmd = [HIPCC, *FLAGS, *EXTRA.get(os.path.basename(src), []), "-c", src, "-o", obj]
        cmds.append(cmd)
        if asm:   # device assembly next to the objects, for inspection
            cmds.append([HIPCC, *FLAGS, *EXTRA.get(os.path.basename(src), []), "-S", "--offload-device-only",
                         src, "-o", obj[:-2] + ".s"])
    with ThreadPoolExecutor(max_workers=jobs + 1) as ex:
        marshal = ex.submit(build_marshal)
        list(ex.map(_run, cmds))
        marshal.result()
    tmp = LIB + f".{os.getpid()}.tmp"
    _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp])
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(asm="--asm" in sys.argv))
