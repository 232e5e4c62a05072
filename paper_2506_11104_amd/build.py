"""Compile the HIP sources under csrc/ into paper_2506_11104_amd/libdam.so for gfx950, and the Python
extension csrc/py_native.cpp (host code on torch's headers) into paper_2506_11104_amd/_dam_native.so.

hipcc cross-compiles without a GPU. Packed-fp32 code generation is switched off for the device
pass (the host pass does not know the feature and says so; that warning is harmless).
"""
import glob
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libdam.so")
OBJ = os.path.join(HERE, "_build")

FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-fhip-fp32-correctly-rounded-divide-sqrt", "-Wall", "-Wno-unused-function",
         "-Wno-unknown-warning-option", "-Wno-inline-asm"]

# The capture kernels read every accumulator right after its chain of products: with the results in
# ordinary vector registers no copies out of the accumulation registers are needed.
EXTRA = {"dam_capture.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"]}


NATIVE = os.path.join(HERE, "_dam_native.so")


def build_native():
    """The extension links against libdam.so beside it and against the torch that will import it."""
    import sysconfig

    import torch
    t = os.path.dirname(torch.__file__)
    cmd = ["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-I" + os.path.join(ROOT, "include"),
           "-I" + sysconfig.get_paths()["include"], "-isystem", os.path.join(t, "include"), "-isystem",
           os.path.join(t, "include", "torch", "csrc", "api", "include"), "-isystem", "/opt/rocm/include",
           os.path.join(CSRC, "py_native.cpp"), "-o", NATIVE, "-L" + HERE, "-ldam", "-L" + os.path.join(t, "lib"), "-lc10",
           "-lc10_hip", "-ltorch_cpu", "-ltorch_python", "-Wl,-rpath,$ORIGIN"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed for py_native.cpp:\n" + r.stderr)


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build(force: bool = True, verbose: bool = False) -> str:
    srcs = sources()
    deps = srcs + [os.path.join(CSRC, "py_native.cpp")] + glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(ROOT, "include", "*.h"))
    newest = max(os.path.getmtime(f) for f in deps)
    if not force and all(os.path.exists(f) and os.path.getmtime(f) >= newest for f in (OUT, NATIVE)):
        return OUT
    os.makedirs(OBJ, exist_ok=True)

    def compile_one(src):
        obj = os.path.join(OBJ, os.path.basename(src) + ".o")
        cmd = ["hipcc", "-c", src, "-o", obj] + FLAGS + EXTRA.get(os.path.basename(src), [])
        r = subprocess.run(cmd, capture_output=True, text=True)
        err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed for {src}:\n{err}")
        if verbose and err.strip():
            print(err, file=sys.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=4) as ex:
        objs = list(ex.map(compile_one, srcs))
    r = subprocess.run(["hipcc", "-shared", "-fPIC", "--offload-arch=gfx950", "-o", OUT] + objs,
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    build_native()
    return OUT


if __name__ == "__main__":
    print(build(force=True, verbose=True))
