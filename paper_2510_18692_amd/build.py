"""Build libmoga.so (the C-ABI HIP library, gfx950, hipcc) and its torch binding in-tree."""
from __future__ import annotations

import os
import re
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmoga.so")
BENCH_LIB = os.path.join(HERE, "libmoga_bench.so")   # peak microbenchmarks for bench.py only
EXAMPLE = os.path.join(HERE, "c_abi_example")
SOURCES = ["api.hip", "route.hip", "permute.hip", "attn_fwd.hip", "attn_bwd.hip", "balance.hip", "static_index.hip"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=default",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # no packed-fp32 VALU ops
    "-Wno-unused-command-line-argument", "-Wno-deprecated-volatile",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    raise RuntimeError("hipcc not found")


def native_path() -> str:
    """The native half of the Python binding.  It follows the ABI of one torch and one interpreter: the name says which,
    so that another one in the same tree gets a file of its own."""
    import torch
    tag = re.sub(r"[^A-Za-z0-9.]+", "_", f"{torch.__version__}-{sysconfig.get_config_var('SOABI')}")
    return os.path.join(HERE, f"_moga_torch-{tag}.so")


def build_native() -> str:
    """Host code only (g++ and torch's headers): the torch binding of the C ABI, against this interpreter's torch."""
    import torch
    from torch.utils import cpp_extension as ext
    path = native_path()
    tmp = f"{path}.{os.getpid()}"   # processes that find it missing at the same time each move a whole file into place
    inc = [ROOT + "/include", *ext.include_paths("cuda"), sysconfig.get_paths()["include"]]
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-DTORCH_EXTENSION_NAME=_moga_torch", "-D__HIP_PLATFORM_AMD__=1",
           "-DUSE_ROCM=1", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *(x for i in inc for x in ("-isystem", i)),
           os.path.join(CSRC, "torch_binding.cpp"), "-o", tmp, "-L", HERE, "-lmoga", "-Wl,-rpath,$ORIGIN",
           *(x for p in ext.library_paths("cuda") for x in ("-L", p)), "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("native binding build failed:\n" + r.stdout + r.stderr)
    os.replace(tmp, path)
    return path


def build(verbose: bool = False, extra_flags=()) -> str:
    """Compile every source and link the shared library.  Always recompiles."""
    hipcc = _hipcc()
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)

    def compile_one(src):
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        cmd = [hipcc, *FLAGS, *extra_flags, "-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        out = "\n".join(l for l in (r.stdout + r.stderr).splitlines()
                        if "packed-fp32-ops" not in l and l.strip())
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed for {src}:\n{out}")
        if verbose and out:
            print(out, file=sys.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout + r.stderr)
    build_native()
    # the two peak microbenchmarks bench.py reports beside the published peaks (a library of their own)
    r = subprocess.run([hipcc, *FLAGS, *extra_flags, "-shared", os.path.join(CSRC, "bench_peaks.hip"),
                        "-o", BENCH_LIB], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("bench library build failed:\n" + r.stdout + r.stderr)
    # a torch-free client of the C ABI (run by the GPU tests)
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-O2", "-I", os.path.join(ROOT, "include"),
                        os.path.join(CSRC, "c_abi_example.cpp"), "-L", HERE, "-lmoga", "-Wl,-rpath,$ORIGIN",
                        "-o", EXAMPLE], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("example build failed:\n" + r.stdout + r.stderr)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
