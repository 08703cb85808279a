"""Build libsbnet_hip.so for gfx950 with hipcc (cross-compiles without a GPU) and _torch_calls.so, the host code that
takes torch tensors to its C ABI."""
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsbnet_hip.so")
CALLS = os.path.join(HERE, "_torch_calls.so")
OBJ = os.path.join(HERE, "_build")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed fp32 instructions stay off on this target
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


def _compile(src):
    obj = os.path.join(OBJ, os.path.basename(src)[:-4] + ".o")
    cmd = ["hipcc", *HIPCC_FLAGS, "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, err))
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _compile_calls():
    """Host code only: g++, against the headers and libraries of the installed torch."""
    import torch
    base = os.path.dirname(torch.__file__)
    inc = [os.path.join(base, "include"), os.path.join(base, "include", "torch", "csrc", "api", "include"),
           os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"), sysconfig.get_paths()["include"]]
    obj = os.path.join(OBJ, "torch_calls.o")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-DUSE_ROCM", "-D__HIP_PLATFORM_AMD__",
                           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch.compiled_with_cxx11_abi()), "-Wall",
                           *["-isystem" + d for d in inc], "-c", os.path.join(CSRC, "torch_calls.cpp"), "-o", obj])
    return obj, os.path.join(base, "lib")


def _link_calls(obj, torch_lib):
    # the library itself is found beside this one; torch's are loaded by `import torch` already
    subprocess.check_call(["g++", "-shared", "-o", CALLS, obj, "-L" + HERE, "-l:libsbnet_hip.so", "-L" + torch_lib, "-lc10",
                           "-lc10_hip", "-ltorch_cpu", "-ltorch_python", "-Wl,-rpath,$ORIGIN"])


def build(verbose=False):
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=4) as ex:
        calls = ex.submit(_compile_calls)
        objs = list(ex.map(_compile, sources()))
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    subprocess.check_call(cmd)
    _link_calls(*calls.result())
    if verbose:
        print("built", LIB, CALLS)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
