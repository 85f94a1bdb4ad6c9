"""Build libsqmi.so (HIP, gfx950 only) and the binding's native calls in-tree next to the sources."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libsqmi.so")
TILE_SOURCES = [f"gemm_i8_tile_{layout}{output}.hip" for layout in ("rows", "tiled") for output in ("", "_ragged", "_codes")]
SOURCES = ["api.hip", "quantize.hip", "weight_prep.hip", "rowops.hip", "gemm_i8.hip", *TILE_SOURCES, "gemm_i8_stream.hip", "gemm_i8_direct.hip", "gemm_i8_direct_rows.hip", "gemm_i8_direct_tiled.hip", "bmm_strip.hip", "bmm_pv.hip", "attn_fused.hip", "attn_few.hip", "probe.hip"]

# -ffp-contract=off: scale arithmetic must round every product and sum separately (bit-exact codes).
# packed-fp32 ops are disabled for the whole library.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off", "-fno-fast-math",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall", "-Wno-unused-function",
         "-I", INCLUDE, "-I", CSRC]
# Tiles with one wave per SIMD: MFMAs on plain vector registers, accumulation registers only for what does not fit (gemm_tile.h).  The other tiles of
# these files run with the option as without it (times with / without it, means over ten to twenty calls of each: tiles of 32, 64 and 128 rows
# 0.99, 0.98 and 0.97, of 256 x 192 1.00, x 256 1.00 and 1.01, x 384 1.00 and 1.01, of 128 x 128 1.00).
FLAGS_OF = {src: ["-mllvm", "-amdgpu-mfma-vgpr-form=true"] for src in TILE_SOURCES}


def build_host_calls() -> str:
    """The native form of the binding's common calls (host code only, against the installed torch).  Always recompiles."""
    import sysconfig

    import torch
    root = os.path.dirname(torch.__file__)
    out = os.path.join(HERE, "_host_calls.so")
    inc = [INCLUDE, os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"), sysconfig.get_paths()["include"],
           os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")]
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-w", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM",
                    f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *(a for i in inc for a in ("-I", i)),
                    os.path.join(CSRC, "host_calls.cpp"), "-o", out, "-L", os.path.join(root, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python",
                    f"-Wl,-rpath,{os.path.join(root, 'lib')}"], check=True)
    return out


def build(verbose: bool = False, jobs: int = 8) -> str:
    """Compile every source and link the shared library.  Always recompiles."""
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs = []
    objs = []
    for src in SOURCES:
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        objs.append(obj)
        cmd = ["hipcc", *FLAGS, *FLAGS_OF.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    failed = False
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l and l.strip())
        if p.returncode != 0:
            failed = True
            print(f"[build] {src} FAILED\n{out}", file=sys.stderr)
        elif verbose and out:
            print(out)
    if failed:
        raise RuntimeError("hipcc failed")
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs], check=True)
    build_host_calls()
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
