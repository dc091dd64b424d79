"""Build libqbert.so (the C-ABI HIP library) for gfx950 with hipcc, and the Python binding's native half _calls.so (host
code against torch's headers and libqbert.so) with the host compiler, in-tree."""
import os
import subprocess
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libqbert.so")
CALLS = os.path.join(HERE, "_calls.so")
SOURCES = ("api.hip", "quantize.hip", "qgemm_i8.hip", "qgemm_i8_list.hip", "bwd_bf16.hip", "bwd_direct.hip", "hessian.hip")
# packed-fp32 instructions are switched off for every device translation unit
COMMON = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wno-inline-asm",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
# the quantizers (also the one in the GEMM's 8-bit-output epilogue) need one rounding per operation: no fused
# multiply-add contraction there.  (__fmul_rn/__fadd_rn are plain operators to the compiler and would be fused.)
PER_FILE = {"quantize.hip": ["-ffp-contract=off"], "qgemm_i8.hip": ["-ffp-contract=off"], "qgemm_i8_list.hip": ["-ffp-contract=off"]}


def compile_calls(verbose=False):
    """The object file of the binding's native half; linked against libqbert.so afterwards."""
    import torch
    inc = os.path.join(os.path.dirname(torch.__file__), "include")
    obj = os.path.join(CSRC, "host_calls.o")
    # (the two definitions select the HIP side of torch's own headers)
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-w", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, "-I/opt/rocm/include", "-I" + inc,
           "-I" + os.path.join(inc, "torch", "csrc", "api", "include"), "-I" + sysconfig.get_paths()["include"],
           "-c", os.path.join(CSRC, "host_calls.cpp"), "-o", obj]
    if verbose:
        print(" ".join(cmd))
    subprocess.run(cmd, check=True)
    return obj


def link_calls(obj):
    import torch
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = ["g++", "-shared", obj, "-o", CALLS, "-L" + lib, "-ltorch_python", "-ltorch_cpu", "-ltorch_hip", "-lc10", "-lc10_hip",
           "-L" + HERE, "-l:libqbert.so", "-Wl,-rpath,$ORIGIN"]
    subprocess.run(cmd, check=True)
    os.remove(obj)


def build(verbose=False):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    def compile_one(src):
        obj = os.path.join(CSRC, src.replace(".hip", ".o"))
        cmd = [hipcc] + COMMON + PER_FILE.get(src, []) + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd))
        subprocess.run(cmd, check=True, stderr=None if verbose else subprocess.DEVNULL)
        return obj

    with ThreadPoolExecutor(max_workers=min(len(SOURCES) + 1, 8)) as pool:   # one translation unit per worker
        calls = pool.submit(compile_calls, verbose)
        objs = list(pool.map(compile_one, SOURCES))
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", LIB]
    subprocess.run(cmd, check=True)
    for o in objs:
        os.remove(o)
    link_calls(calls.result())
    return LIB


if __name__ == "__main__":
    print("built", build(verbose=True))
