"""Builds libpolarquant.so (the HIP kernels and their C ABI) for gfx950, and the Python binding's
native part (_native.<ABI tag>.so), in-tree.  The latter is host code that only makes calls cheaper: where a compiler
or the headers for it are missing the build says so and goes on.

`python -m paper_2502_00527_amd.build` compiles every source under csrc/ with
hipcc; it cross-compiles without a GPU.  The flags matter for correctness:
floating-point contraction is off (the encoder's fp32/fp64 operation chains are
part of the definition of the codes; fused multiply-adds are written out where
wanted), and packed-fp32 instructions are disabled.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
LIB_PATH = os.path.join(PKG_DIR, "libpolarquant.so")
SOURCES = ["pq_api.hip", "pq_encode.hip", "pq_values.hip", "pq_decode.hip", "pq_decode_matrix.hip", "pq_decode_matrix_v4.hip", "pq_decode_matrix_v2.hip",
           "pq_decode_partials_ga.hip", "pq_decode_grouped.hip", "pq_decode_grouped_v4.hip", "pq_decode_grouped_v2.hip"]

# the Python binding's argument marshalling (host code only), named for the interpreter it is built for
BINDING = "pq_binding.cpp"
BINDING_PATH = os.path.join(PKG_DIR, "_native" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found; libpolarquant needs the ROCm toolchain")
    return exe


def _filter(text: str) -> str:
    return "\n".join(l for l in text.splitlines()
                     if "packed-fp32-ops" not in l and "is not a recognized feature" not in l)


def binding_lacks():
    """What the binding cannot be built without and is not there; None if it can be."""
    if shutil.which("g++") is None:
        return "g++"
    python_h = os.path.join(sysconfig.get_paths()["include"], "Python.h")
    if not os.path.exists(python_h):
        return python_h
    try:
        from torch.utils import cpp_extension
    except ImportError as e:
        return str(e)
    header = os.path.join("torch", "csrc", "autograd", "python_variable.h")
    if not any(os.path.exists(os.path.join(d, header)) for d in cpp_extension.include_paths()):
        return header
    return None


def _binding_commands(inc, obj):
    """Compile and link commands of the binding; it finds libpolarquant.so beside itself."""
    import torch
    from torch.utils import cpp_extension
    torch_inc = [f for d in cpp_extension.include_paths() for f in ("-isystem", d)]
    abi = [f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DPQ_TORCH_VERSION="{torch.__version__}"']
    compile_ = ["g++", "-O2", "-std=c++17", "-fPIC", "-Wall", *abi, *inc, *torch_inc, "-isystem", sysconfig.get_paths()["include"],
                "-c", os.path.join(CSRC, BINDING), "-o", obj]
    link = ["g++", "-shared", obj, "-o", BINDING_PATH, "-L", PKG_DIR, "-lpolarquant", "-Wl,-rpath,$ORIGIN",
            *[f for d in cpp_extension.library_paths() for f in ("-L", d)], "-ltorch_python", "-ltorch_cpu", "-lc10"]
    return compile_, link


def build(verbose: bool = True, extra_flags=()) -> str:
    """Compiles every translation unit (in parallel) and links libpolarquant.so and the binding."""
    obj_dir = os.path.join(PKG_DIR, "_build")
    os.makedirs(obj_dir, exist_ok=True)
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    procs = []
    for src in SOURCES:
        obj = os.path.join(obj_dir, src.replace(".hip", ".o"))
        cmd = [hipcc(), *FLAGS, *extra_flags, *inc, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, obj, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for name in os.listdir(PKG_DIR):                       # of an earlier build, or of one for another interpreter
        if name.startswith("_native.") and name.endswith(".so"):
            os.unlink(os.path.join(PKG_DIR, name))
    binding, lacks = None, binding_lacks()
    if lacks is None:
        compile_, link_binding = _binding_commands(inc, os.path.join(obj_dir, BINDING.replace(".cpp", ".o")))
        if verbose:
            print(" ".join(compile_), flush=True)
        binding = subprocess.Popen(compile_, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    else:
        print(f"{BINDING} is not built ({lacks} is missing): calls are marshalled by ctypes", file=sys.stderr, flush=True)
    objs = []
    for src, obj, proc in procs:
        out, _ = proc.communicate()
        if proc.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n" + _filter(out))
        if verbose and _filter(out).strip():
            print(_filter(out))
        objs.append(obj)
    link = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB_PATH]
    if verbose:
        print(" ".join(link), flush=True)
    res = subprocess.run(link, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("link failed:\n" + _filter(res.stdout + res.stderr))
    if binding is None:
        return LIB_PATH
    out, _ = binding.communicate()
    if binding.returncode != 0:
        raise RuntimeError(f"g++ failed on {BINDING}:\n{out}")
    res = subprocess.run(link_binding, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("link of the binding failed:\n" + res.stdout + res.stderr)
    return LIB_PATH


if __name__ == "__main__":
    build()
    sys.exit(0)
