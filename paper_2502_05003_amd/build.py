"""Builds libquest.so (the C-ABI HIP library) in-tree with hipcc for gfx950, and the binding's native part."""
from __future__ import annotations

import os
import subprocess
import sysconfig

_HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(_HERE, "csrc")
LIB = os.path.join(_HERE, "libquest.so")
# binding.py's calls in native code (csrc/python_calls.cpp), for one interpreter, which its name tells, and one torch
PYTHON_LIB = os.path.join(_HERE, "quest_python" + sysconfig.get_config_var("EXT_SUFFIX"))
PROBE_LIB = os.path.join(_HERE, "libquest_probe.so")   # measurement aid of bench.py (include/quest_probe.h)
SOURCES = ["quest_api.hip", "hadamard_quantize.hip", "hadamard_quantize_mfma.hip", "hadamard_quantize_rows.hip",
           "lowbit_gemm.hip", "skinny_gemm.hip", "fp4_gemm.hip", "trust_backward.hip", "trust_backward_mfma.hip",
           "trust_backward_rows.hip", "grad_gemm.hip",
           "grad_gemm_mid.hip"]
# per-source extra flags: kernels whose MFMA results are consumed by vector code keep them in VGPRs
EXTRA_FLAGS = {"hadamard_quantize_mfma.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
               "hadamard_quantize_rows.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
               "trust_backward_rows.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
               "trust_backward_mfma.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]}
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
    # packed fp32 VALU forms stay off: plain fp32 ops only
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


def python_calls_command(out: str) -> list[str]:
    """The CPython module: host code against the headers and libraries of the installed torch."""
    import torch

    from .binding import torch_build
    root = os.path.dirname(torch.__file__)
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DQUEST_TORCH_BUILD="{torch_build()}"',
            "-I" + sysconfig.get_paths()["include"],
            "-I" + os.path.join(root, "include"), "-I" + os.path.join(root, "include", "torch", "csrc", "api", "include"),
            os.path.join(CSRC, "python_calls.cpp"), "-o", out, "-L" + os.path.join(root, "lib"), "-ltorch_python",
            "-ltorch_cpu", "-lc10", "-Wl,-rpath," + os.path.join(root, "lib")]


def build_python_calls() -> bool:
    """Compiles the CPython module; without a compiler or Python's headers there is none, and calls go through ctypes."""
    tmp = PYTHON_LIB + f".tmp{os.getpid()}"
    cmd = python_calls_command(tmp)
    try:
        run = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
        built, why = run.returncode == 0, run.stdout.decode()
    except OSError as error:
        built, why = False, str(error)
    if built:
        os.replace(tmp, PYTHON_LIB)
    else:
        print("quest_python was not built, calls from Python take 3 us more: " + " ".join(cmd) + "\n" + why)
        if os.path.exists(PYTHON_LIB):
            os.remove(PYTHON_LIB)   # that of another build
    return built


def build_library(verbose: bool = False) -> str:
    """Compile every source and link libquest.so; always recompiles."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(_HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs = []
    objects = []
    for src in SOURCES:
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        objects.append(obj)
        cmd = [hipcc, *HIPCC_FLAGS, *EXTRA_FLAGS.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
        procs.append((cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)))
    build_python_calls()
    for cmd, proc in procs:
        out = proc.communicate()[0].decode()
        lines = [l for l in out.splitlines() if "not a recognized feature" not in l]
        if proc.returncode != 0:
            raise RuntimeError("compilation failed: " + " ".join(cmd) + "\n" + "\n".join(lines))
        if verbose and lines:
            print("\n".join(lines))
    tmp = LIB + f".tmp{os.getpid()}"
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objects])
    os.replace(tmp, LIB)
    tmp = PROBE_LIB + f".tmp{os.getpid()}"
    out = subprocess.run([hipcc, *HIPCC_FLAGS, "-shared", os.path.join(CSRC, "peak_probe.hip"), "-o", tmp],
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    if out.returncode != 0:
        raise RuntimeError("hipcc failed on peak_probe.hip\n" + out.stdout.decode())
    os.replace(tmp, PROBE_LIB)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
