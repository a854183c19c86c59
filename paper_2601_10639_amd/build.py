"""Builds libstem.so in-tree with hipcc for gfx950 (cross-compiles without a GPU)."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libstem.so")
BIND = os.path.join(HERE, "_bind.so")   # the hot calls' binding, a Python module
OBJ_DIR = os.path.join(HERE, "_build")
SOURCES = ["api.hip", "gemm_bf16.hip", "gemm_skinny_bf16.hip", "gemm_decode_bf16.hip", "ffn_decode_bf16.hip", "kernels_f32.hip", "embed_grad.hip", "embed_grad_static.hip", "adamw.hip", "prefetch.hip", "edit.hip", "calibrate.hip"]
FLAGS = ["-O3", "--offload-arch=gfx950", "-fPIC", "-std=c++17",
         # keep the compiler from forming packed-fp32 instructions
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    return "hipcc"


def _run(cmd):
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError("command failed: %s\n%s\n%s" % (" ".join(cmd), r.stdout, err))
    return err


def _build_bind() -> str:
    import sysconfig

    import torch
    from torch.utils import cpp_extension

    inc = [f"-I{p}" for p in (*cpp_extension.include_paths(), sysconfig.get_paths()["include"])]
    torch_lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    obj = os.path.join(OBJ_DIR, "bind.o")
    msg = _run(["g++", "-O2", "-fPIC", "-std=c++17", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *inc,
                "-c", os.path.join(CSRC, "bind.cpp"), "-o", obj])
    # (libstem.so is found beside it; torch's libraries are loaded by then)
    _run(["g++", "-shared", "-o", BIND, obj, f"-L{HERE}", "-l:libstem.so", "-Wl,-rpath,$ORIGIN", f"-L{torch_lib}", "-lc10", "-ltorch_cpu",
          "-ltorch_python"])
    return msg


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    hipcc = _hipcc()
    objs = [os.path.join(OBJ_DIR, s.replace(".hip", ".o")) for s in SOURCES]
    cmds = [[hipcc, *FLAGS, "-c", os.path.join(CSRC, s), "-o", o] for s, o in zip(SOURCES, objs)]
    with ThreadPoolExecutor(max_workers=min(8, len(cmds))) as ex:
        for msg in ex.map(_run, cmds):
            if verbose and msg.strip():
                print(msg, file=sys.stderr)
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs])
    msg = _build_bind()
    if verbose and msg.strip():
        print(msg, file=sys.stderr)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
