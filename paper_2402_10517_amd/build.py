"""Build the HIP library in-tree: paper_2402_10517_amd/libapgemv.so (gfx950 only), and the binding's native calls next to it."""
import os
import subprocess
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libapgemv.so")
TORCH_CALL = os.path.join(HERE, "_torch_call.so")   # Python module; host code only
SOURCES = ["gemv_alu.hip", "gemv_quad.hip", "gemv_matrix.hip", "gemv_tile.hip", "dequant.hip", "gemm_fused.hip", "gemm_static.hip", "dispatch.cpp", "api.cpp", "pack.cpp",
           "dense_gemm.cpp", "quantize.cpp"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument"]


def build(verbose=False):
    """Compile every source to an object file (in parallel, one hipcc per file), then link."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ, exist_ok=True)

    def compile_one(name):
        obj = os.path.join(OBJ, name + ".o")
        cmd = [hipcc] + FLAGS + ["-x", "hip", "-c", os.path.join(CSRC, name), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
        return obj

    def compile_torch_call():
        import torch
        base = os.path.dirname(torch.__file__)
        obj = os.path.join(OBJ, "torch_call.o")
        cmd = [hipcc, "-x", "c++", "-O2", "-std=c++17", "-fPIC", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", "-I" + os.path.join(base, "include"),
               "-I" + os.path.join(base, "include", "torch", "csrc", "api", "include"), "-I" + sysconfig.get_paths()["include"],
               "-I/opt/rocm/include", "-Wno-unused-command-line-argument", "-c", os.path.join(CSRC, "torch_call.cpp"), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
        return obj, os.path.join(base, "lib")

    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES) + 1)) as pool:
        torch_call = pool.submit(compile_torch_call)
        objs = list(pool.map(compile_one, SOURCES))
        torch_call, torch_lib = torch_call.result()
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", LIB, "-ldl"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    # torch's libraries are loaded by the time the module is; the library above is found next to it
    cmd = [hipcc, "-shared", "-fPIC", torch_call, "-o", TORCH_CALL, "-L" + HERE, "-l:libapgemv.so", "-Wl,-rpath,$ORIGIN", "-L" + torch_lib,
           "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
