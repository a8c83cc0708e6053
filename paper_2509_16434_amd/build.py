"""Builds libppo_learner.so (HIP, gfx950, hipcc) and the native part of its Python binding (_binding.so, g++) in-tree."""
from __future__ import annotations

import os
import subprocess
import sysconfig

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(_HERE, "libppo_learner.so")
SRC = os.path.join(_HERE, "csrc", "ppo_learner.hip")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def sources():
    d = os.path.join(_HERE, "csrc")
    inc = os.path.join(os.path.dirname(_HERE), "include")
    return [os.path.join(d, f) for f in sorted(os.listdir(d))] + [os.path.join(inc, f) for f in sorted(os.listdir(inc))]


BINDING = os.path.join(_HERE, "_binding.so")
BINDING_SRC = os.path.join(_HERE, "csrc", "binding.cpp")
CXX = os.environ.get("CXX", "g++")


def binding_command():
    import torch
    from torch.utils import cpp_extension
    inc = [p for p in cpp_extension.include_paths() if "hip" not in os.path.basename(p)] + [sysconfig.get_paths()["include"]]
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    return ([CXX, "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"] + [x for p in inc for x in ("-isystem", p)] +
            [BINDING_SRC, "-o", BINDING, f"-L{lib}", "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", f"-Wl,-rpath,{lib}"])


def stale() -> bool:
    if not (os.path.exists(LIB) and os.path.exists(BINDING)):
        return True
    t = min(os.path.getmtime(LIB), os.path.getmtime(BINDING))
    return any(os.path.getmtime(s) > t for s in sources())


def build_lib(force: bool = True, verbose: bool = False) -> str:
    """Compile the library and the binding, side by side; with force=False only when a source is newer than they are."""
    if force or stale():
        cmds = {"hipcc": [HIPCC] + FLAGS + ["-o", LIB, SRC], CXX: binding_command()}
        if verbose:
            for cmd in cmds.values():
                print(" ".join(cmd))
        runs = {n: subprocess.Popen(cmd, stdout=subprocess.DEVNULL, stderr=subprocess.PIPE, text=True) for n, cmd in cmds.items()}
        # every process is read to its end before any failure is reported: one left with a full pipe never ends
        errs = {n: "\n".join(l for l in r.communicate()[1].splitlines() if "packed-fp32-ops" not in l) for n, r in runs.items()}
        failed = [f"{n} failed:\n{errs[n]}" for n, r in runs.items() if r.returncode != 0]
        if failed:
            raise RuntimeError("\n".join(failed))
        if verbose:
            for err in errs.values():
                if err.strip():
                    print(err)
    return LIB


if __name__ == "__main__":
    print(build_lib(True, True))
