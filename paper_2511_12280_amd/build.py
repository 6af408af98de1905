"""Build libd3tom.so (HIP, gfx950; hipcc) and the extension that binds it (g++), in-tree.  `python -m paper_2511_12280_amd.build`."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libd3tom.so")
NATIVE = os.path.join(HERE, "_native.so")
SOURCES = ["api.hip", "importance.hip", "topk.hip", "merge.hip", "attend.hip", "deciders.hip", "linear.hip", "block_ops.hip",
           "stack.hip", "pipeline.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # no packed-fp32 VALU forms
         "-mllvm", "-amdgpu-kernarg-preload-count=16",                  # first arguments arrive in registers: one load less in front of every kernel
         "-Wall", "-Wno-unused-function"]


def source_digest() -> str:
    """Short digest of the kernel sources (every file under csrc/ and the C header): lets a stored measurement say
    which sources it was taken on."""
    import hashlib
    h = hashlib.sha256()
    files = sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith((".hip", ".hpp")))
    files.append(os.path.join(os.path.dirname(HERE), "include", "d3tom.h"))
    for f in files:
        h.update(os.path.basename(f).encode())
        h.update(open(f, "rb").read())
    return h.hexdigest()[:16]


def build(verbose: bool = False) -> str:
    cmd = ["hipcc"] + FLAGS + [os.path.join(CSRC, s) for s in SOURCES] + ["-o", LIB]
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + err)
    if verbose and err.strip():
        print(err, file=sys.stderr)
    build_native()
    return LIB


def build_native() -> str:
    """The extension between Python and libd3tom.so (g++, against the installed torch's headers)."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"]
    cmd += ["-isystem" + d for d in cpp_extension.include_paths() + [sysconfig.get_paths()["include"]]]
    cmd += [os.path.join(CSRC, "native.cpp"), "-L" + HERE, "-l:libd3tom.so"]
    cmd += ["-L" + d for d in cpp_extension.library_paths()] + ["-lc10", "-ltorch_cpu", "-ltorch", "-ltorch_python"]
    res = subprocess.run(cmd + ["-Wl,-rpath,$ORIGIN", "-o", NATIVE], capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("g++ failed:\n" + res.stderr)
    return NATIVE


if __name__ == "__main__":
    print(build(verbose=True))
