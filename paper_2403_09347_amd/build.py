"""Builds libburst.so (the C-ABI library) from csrc/ with hipcc for gfx950, in-tree, and beside it the
torch module of the differentiable call (host code only, against the installed torch)."""
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libburst.so")
SOURCES = ["burst_api.hip", "burst_elementwise.hip", "burst_generic.hip",
           "burst_fwd_mfma.hip", "burst_bwd_dq_mfma.hip", "burst_bwd_dkv_mfma.hip",
           "burst_materialized.hip", "burst_d64_mfma.hip", "burst_d128_plain.hip",
           "burst_d32_pad.hip", "burst_d64_pad.hip", "burst_d96_pad.hip", "burst_d128_pad.hip", "burst_probe.hip"]
FLAGS = ["-O3", "--offload-arch=gfx950", "-fPIC", "-std=c++17", "-ffast-math", "-fno-finite-math-only", "-fno-honor-nans",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-mllvm", "-amdgpu-mfma-vgpr-form=1", "-Wno-unused-command-line-argument",
         "-Wno-inline-asm"]   # the DMA helper names M0 as clobbered, which the compiler reports as a reserved register


TORCH_SRC = "burst_torch.cpp"
TORCH_LIB = os.path.join(HERE, "_burst_torch.so")


def _torch_commands():
    """Compile and link command of the torch module."""
    import torch
    from torch.utils import cpp_extension
    cxx = os.environ.get("CXX", "g++")
    obj = os.path.join(HERE, "_build", TORCH_SRC.replace(".cpp", ".o"))
    include = cpp_extension.include_paths() + [sysconfig.get_paths()["include"], "/opt/rocm/include"]
    compile_cmd = [cxx, "-O2", "-fPIC", "-std=c++17", "-DUSE_ROCM=1", "-D__HIP_PLATFORM_AMD__=1",
                   "-DTORCH_API_INCLUDE_EXTENSION_H", "-DTORCH_EXTENSION_NAME=_burst_torch",
                   f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
                   *[x for d in include for x in ("-isystem", d)], "-c", os.path.join(CSRC, TORCH_SRC), "-o", obj]
    link_cmd = [cxx, "-shared", obj, "-o", TORCH_LIB, *["-L" + d for d in cpp_extension.library_paths()], "-lc10", "-lc10_hip",
                "-ltorch", "-ltorch_cpu", "-ltorch_hip", "-ltorch_python", "-L" + HERE, "-lburst", "-Wl,-rpath,$ORIGIN"]
    return compile_cmd, link_cmd


def build(verbose=True, jobs=8):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs, procs = [], []
    os.makedirs(os.path.join(HERE, "_build"), exist_ok=True)
    torch_compile, torch_link = _torch_commands()
    if verbose:
        print(" ".join(torch_compile), flush=True)
    procs.append((TORCH_SRC, subprocess.Popen(torch_compile, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for src in SOURCES:
        obj = os.path.join(HERE, "_build", src.replace(".hip", ".o"))
        objs.append(obj)
        cmd = [hipcc, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        if len(procs) >= jobs:
            _drain(procs, verbose)
    _drain(procs, verbose)
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    if verbose:
        print(" ".join(torch_link), flush=True)
    subprocess.run(torch_link, check=True)
    build_example(verbose)
    return LIB


EXAMPLE_SRC = os.path.join(HERE, "examples", "ring_walk.cpp")
EXAMPLE_BIN = os.path.join(HERE, "_build", "ring_walk")


def build_example(verbose=True):
    """The plain host program that walks a ring share through the C ABI (no Python on its path),
    linked against the library just built; run by tests/test_gpu_c_example.py."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, "-O2", "-std=c++17", "--offload-arch=gfx950", "-I", os.path.join(os.path.dirname(HERE), "include"),
           EXAMPLE_SRC, "-L", HERE, "-lburst", "-Wl,-rpath,$ORIGIN/..", "-o", EXAMPLE_BIN]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return EXAMPLE_BIN


def _drain(procs, verbose):
    while procs:
        src, p = procs.pop(0)
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            sys.stderr.write(out + "\n")
            raise RuntimeError("compilation failed: " + src)
        if verbose and out.strip():
            print(out)


if __name__ == "__main__":
    build()
