"""Build libsignsgd.so (the C-ABI HIP library) for gfx950 and the Python module
that marshals torch tensors into it, in-tree.

    python -m paper_1802_04434_amd.build

Flags: FP contraction off (momentum must round each product and the sum
separately), packed-fp32 instructions disabled, no fast-math.
"""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsignsgd.so")
SOURCES = ["api.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off", "-fno-fast-math",
    "-fno-gpu-flush-denormals-to-zero",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def build(out=LIB, verbose=False):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = out + ".tmp%d" % os.getpid()
    cmd = [hipcc, *HIPCC_FLAGS, "-o", tmp] + [os.path.join(CSRC, s) for s in SOURCES]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, out)
    return out


MARSHAL = os.path.join(HERE, "_marshal.so")


def build_marshal(verbose=False):
    """The CPython module between torch tensors and the library (csrc/marshal.cpp): plain host C++
    against torch's headers; it finds libsignsgd.so next to itself."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    tmp = MARSHAL + ".tmp%d" % os.getpid()
    torch_lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI)]
    for inc in cpp_extension.include_paths() + [os.path.join(rocm, "include"), sysconfig.get_paths()["include"]]:
        cmd += ["-isystem", inc]
    cmd += [os.path.join(CSRC, "marshal.cpp"), "-o", tmp, "-L" + HERE, "-lsignsgd", "-L" + torch_lib, "-ltorch_python",
            "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip", "-L" + os.path.join(rocm, "lib"), "-lamdhip64",
            "-Wl,-rpath,$ORIGIN"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, MARSHAL)
    return MARSHAL


ABI_CHECK = os.path.join(HERE, "abi_check")


def build_abi_check(verbose=False):
    """The stand-alone C++ host program that drives the library without Python
    (csrc/abi_check.cpp); it finds libsignsgd.so next to itself."""
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    tmp = ABI_CHECK + ".tmp%d" % os.getpid()
    # plain host C++: only the HIP runtime API (hipMalloc, hipMemcpy, streams) and the library
    cmd = ["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(rocm, "include"),
           os.path.join(CSRC, "abi_check.cpp"), "-o", tmp, "-L" + HERE, "-lsignsgd",
           "-L" + os.path.join(rocm, "lib"), "-lamdhip64", "-Wl,-rpath,$ORIGIN", "-Wl,-rpath," + os.path.join(rocm, "lib")]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, ABI_CHECK)
    return ABI_CHECK


if __name__ == "__main__":
    print(build(verbose=True))
    print(build_marshal(verbose=True))
    print(build_abi_check(verbose=True))
