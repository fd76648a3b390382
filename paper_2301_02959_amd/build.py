"""Builds libflexshard_hip.so for gfx950 with hipcc (cross-compiles without a GPU), and the binding's native helper."""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libflexshard_hip.so")
# named for the interpreter, so that no other one loads it
MARSHAL = os.path.join(PKG, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))
UNTAGGED = os.path.join(PKG, "_marshal.so")                # what any interpreter would load in its place

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off",                                   # every float add stays one IEEE operation
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # no packed-fp32 instructions
    "-Wall", "-Wno-unused-function",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    deps = sources() + glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(ROOT, "include", "*.h"))
    return any(os.path.getmtime(p) > t for p in deps)


def helper_stale() -> bool:
    return not os.path.exists(MARSHAL) or os.path.getmtime(os.path.join(CSRC, "marshal.cpp")) > os.path.getmtime(MARSHAL)


def helper_command(out):
    """The binding's native helper (no device code): against the installed torch's own headers and libraries."""
    import torch
    base = os.path.dirname(torch.__file__)
    built_for = f"{torch.__version__} {torch.version.git_version}"
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", os.path.join(CSRC, "marshal.cpp"),
            "-I", os.path.join(base, "include"), "-I", os.path.join(base, "include", "torch", "csrc", "api", "include"),
            "-I", sysconfig.get_paths()["include"], f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            f'-DFS_BUILT_FOR="{built_for}"',
            "-L", os.path.join(base, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-o", out]


def build_helper(verbose: bool = False) -> bool:
    """The library and the package do without the helper (the binding then checks its pointers in Python), so a machine
    without a host compiler or torch's headers is told so and goes on; no helper of another source stays behind."""
    out = MARSHAL + ".new"
    try:
        cmd = helper_command(out)
        if verbose:
            print(" ".join(cmd), flush=True)
        done = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        said = done.stdout.strip()
        built = done.returncode == 0 and os.path.exists(out)
    except OSError as e:
        said, built = str(e), False
    if said:
        print(said, file=sys.stderr)
    if built:
        os.replace(out, MARSHAL)
        if os.path.exists(UNTAGGED):
            os.remove(UNTAGGED)
        return True
    for path in (out, MARSHAL, UNTAGGED):
        if os.path.exists(path):
            os.remove(path)
    print("marshal.cpp did not compile: the binding will check its pointers in Python", file=sys.stderr)
    return False


def build_library(verbose: bool = False) -> None:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs = []
    obj_dir = os.path.join(PKG, "_build")
    os.makedirs(obj_dir, exist_ok=True)
    procs = []
    for src in sources():
        obj = os.path.join(obj_dir, os.path.basename(src) + ".o")
        objs.append(obj)
        cmd = [hipcc, *[f for f in FLAGS if f != "-shared"], "-c", src, "-I", os.path.join(ROOT, "include"),
               "-I", CSRC, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    failed = False
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l and l.strip())
        if out:
            print(out, file=sys.stderr)
        if p.returncode != 0:
            failed = True
            print(f"hipcc failed on {src}", file=sys.stderr)
    if failed:
        raise RuntimeError("hipcc failed")
    subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB], check=True)


def build(force: bool = True, verbose: bool = False) -> str:
    if force or stale():
        build_library(verbose)
    if force or helper_stale():
        build_helper(verbose)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose="-v" in sys.argv))
