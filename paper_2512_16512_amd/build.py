"""Build ``libxtc.so`` (the gfx950 kernels and the C ABI) and ``_binding.so``
(its entry points over torch tensors, host code only) in-tree.

Every translation unit of the library is compiled with hipcc for gfx950 only,
with packed-fp32 instruction selection disabled, then linked into one shared
library next to this file; where torch is installed, the binding is compiled
against its headers with hipcc's own clang and linked to the library.  Run ``python paper_2512_16512_amd/build.py`` (a plain script: importing the
package needs the built library) or call ``build()``.
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libxtc.so")
BINDING = os.path.join(HERE, "_binding.so")
OBJDIR = os.path.join(HERE, "_build")

SOURCES = ["gemm_f32.hip", "gemm_bf16.hip", "conv2d_f32.hip", "conv2d_bf16.hip", "xtc_api.cpp"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I" + os.path.join(HERE, "..", "include"),
]


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(OBJDIR, os.path.splitext(src)[0] + ".o")
    lang = ["-x", "hip"] if src.endswith(".cpp") else []
    cmd = [HIPCC] + FLAGS + lang + ["-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s%s" % (src, r.stdout, r.stderr))
    return obj


def _run(cmd, what: str, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("%s failed:\n%s%s" % (what, r.stdout, r.stderr))


# the host compiler of the ROCm installation hipcc belongs to
CXX = os.path.join(os.path.dirname(HIPCC), "amdclang++")


def _compile_binding(verbose: bool) -> str | None:
    try:
        import torch
    except ImportError:
        return None      # the C ABI needs no torch
    inc = os.path.join(os.path.dirname(torch.__file__), "include")
    obj = os.path.join(OBJDIR, "torch_binding.o")
    _run([CXX, "-O2", "-std=c++17", "-fPIC", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
          "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
          "-isystem", inc, "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"),
          "-isystem", os.path.join(os.path.dirname(os.path.dirname(HIPCC)), "include"),
          "-isystem", sysconfig.get_paths()["include"],
          "-c", os.path.join(CSRC, "torch_binding.cpp"), "-o", obj], "torch_binding.cpp", verbose)
    return obj


def _link_binding(obj: str, verbose: bool) -> None:
    # torch's libraries are already loaded when the binding is imported;
    # libxtc.so is found next to it
    import torch
    tmp = BINDING + ".tmp%d" % os.getpid()
    _run([CXX, "-shared", "-o", tmp, obj, "-L" + HERE, "-l:libxtc.so", "-Wl,-rpath,$ORIGIN",
          "-L" + os.path.join(os.path.dirname(torch.__file__), "lib"),
          "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"], "link of _binding.so", verbose)
    os.replace(tmp, BINDING)


def build(verbose: bool = False) -> str:
    os.makedirs(OBJDIR, exist_ok=True)
    with ThreadPoolExecutor(min(len(SOURCES) + 1, os.cpu_count() or 1)) as ex:
        binding = ex.submit(_compile_binding, verbose)
        objs = list(ex.map(lambda s: _compile(s, verbose), SOURCES))
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n%s%s" % (r.stdout, r.stderr))
    os.replace(tmp, LIB)
    binding_obj = binding.result()   # (the library is there, whatever became of the binding)
    if binding_obj is not None:
        _link_binding(binding_obj, verbose)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
