"""Builds libjakiro_verify.so for gfx950 with hipcc and the Python extension _native.so that marshals its calls
(both in-tree, next to this file)."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libjakiro_verify.so")
NATIVE = os.path.join(HERE, "_native.so")
SOURCES = ["api.cpp", "tva_f32.hip", "tva_combine.hip", "accept.hip", "accept_coop.hip", "commit.hip",
           "draft_head.hip", "draft_tree.hip", "stream_gemm.hip", "ring_gemm.hip", "tva_wide.hip", "tva_direct.hip"]
# matrix results in ordinary registers: by default a kernel of more than 256 registers keeps all of them in accumulation
# registers, which the vector unit cannot read (32 moves per tile for the scores of tva_wide.hip)
UNIT_FLAGS = {"tva_wide.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"]}
# kernel arguments in scalar registers when a wave starts: the leading ones, fourteen words at most
PRELOAD = ["-mllvm", "-amdgpu-kernarg-preload-count=14"]
for _unit in ("accept.hip", "accept_coop.hip", "draft_head.hip", "stream_gemm.hip", "ring_gemm.hip"):
    UNIT_FLAGS[_unit] = PRELOAD
MERGES = 7  # tva_bf16.hip is compiled once for each of its merges (JK_MERGE)
# packed-fp32 code generation is switched off for all device code
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-inline-asm",  # the LDS-transfer helper names m0 as clobbered on purpose
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def _run(cmd, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
    if r.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed:\n" + err)
    if verbose and err.strip():
        print(err, file=sys.stderr)


def _native_command(output: str):
    """Host code only: the extension sees torch's C++ headers and the library's C header."""
    import torch
    tdir = os.path.dirname(os.path.abspath(torch.__file__))
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
            "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-isystem", os.path.join(tdir, "include"),
            "-isystem", os.path.join(tdir, "include", "torch", "csrc", "api", "include"), "-isystem", os.path.join(rocm, "include"),
            "-isystem", sysconfig.get_paths()["include"], "-c", os.path.join(CSRC, "native.cpp"), "-o", output], os.path.join(tdir, "lib")


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ, exist_ok=True)
    units = [("tva_bf16.hip", f"tva_bf16_{m}.o", [f"-DJK_MERGE={m}"] + PRELOAD) for m in range(MERGES)]
    units += [(s, os.path.splitext(s)[0] + ".o", UNIT_FLAGS.get(s, [])) for s in SOURCES]
    objects = [os.path.join(OBJ, o) for _, o, _ in units]
    native_obj = os.path.join(OBJ, "native.o")
    native_cmd, torch_lib = _native_command(native_obj)
    jobs = [[hipcc] + FLAGS + defines + ["-x", "hip", "-c", os.path.join(CSRC, s), "-o", os.path.join(OBJ, o)]
            for s, o, defines in units] + [native_cmd]
    with ThreadPoolExecutor(min(8, int(os.environ.get("MAX_JOBS", "8")))) as pool:
        list(pool.map(lambda c: _run(c, verbose), jobs))
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC"] + objects + ["-o", LIB], verbose)
    _run(["g++", "-shared", native_obj, "-o", NATIVE, "-L", HERE, "-ljakiro_verify", "-L", torch_lib, "-lc10", "-lc10_hip",
          "-ltorch_hip", "-ltorch_cpu", "-ltorch", "-ltorch_python", "-lamdhip64", "-Wl,-rpath,$ORIGIN"], verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
