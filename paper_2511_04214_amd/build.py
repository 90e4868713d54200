"""Compile the HIP library for gfx950 (hipcc cross-compiles; no GPU needed) and the binding's native part."""
import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libbrq.so")
BINDING = os.path.join(HERE, "_binding" + sysconfig.get_config_var("EXT_SUFFIX"))
SOURCES = ["brq_api.hip", "rotate_quant.hip", "matrix_rotate_quant.hip", "block_summary.hip", "mxfp4_gemm.hip", "mxfp4_gemm_tiled.hip", "mxfp4_gemm_mid.hip"]
# -ffp-contract=off: the rotation's add/sub/mul sequence is part of the result's definition.
# packed fp32 instructions are kept out of the generated code.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall", "-Wno-unused-function"]


def build_library(verbose=False):
    objs = []
    for src in SOURCES:
        obj = os.path.join(CSRC, src.replace(".hip", ".o"))
        cmd = ["hipcc"] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd))
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed on %s:\n%s" % (src, out))
        if verbose and out.strip():
            print(out)
        objs.append(obj)
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs)
    return LIB


def build_binding(verbose=False):
    """The compiled part of the binding, against the installed torch, whose version it is marked with (host code only)."""
    import torch
    t = os.path.dirname(os.path.abspath(torch.__file__))
    include = [os.path.join(t, "include"), os.path.join(t, "include", "torch", "csrc", "api", "include"),
               sysconfig.get_paths()["include"], "/opt/rocm/include"]
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, '-DBRQ_TORCH="%s"' % torch.__version__] + ["-isystem" + i for i in include]
    cmd += [os.path.join(CSRC, "binding.cpp"), "-o", BINDING, "-L" + os.path.join(t, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    if verbose:
        print(" ".join(cmd))
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed on binding.cpp:\n%s" % r.stdout)
    if verbose and r.stdout.strip():
        print(r.stdout)
    return BINDING


if __name__ == "__main__":
    print(build_library(verbose=True))
    print(build_binding(verbose=True))
