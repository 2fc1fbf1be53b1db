"""Build libfewbit.so (HIP kernels for gfx950 + host fit + C ABI) and _native.so
(the calls on torch tensors, host code linked against it) in-tree.  Where torch
or its headers are missing only the first is built: it needs neither, and a
program that uses include/fewbit.h needs no more.

    python -m paper_2202_00441_amd.build      # or: python paper_2202_00441_amd/build.py

Flags:
  --offload-arch=gfx950         MI355X only, one code path
  -O3, no fast-math             IEEE fp32 semantics, denormals kept
  -packed-fp32-ops disabled     no packed fp32 VALU forms are generated
  kernarg preload               pointers and size arrive in scalar registers with the wave:
                                its first loads wait for no load of their addresses (leading
                                pointers and integers only; none if a structure comes first)
  constexpr steps               the bf16 output factors are evaluated at compile time
"""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libfewbit.so")
SOURCES = [os.path.join(CSRC, "fewbit.hip"), os.path.join(CSRC, "fit.cpp")]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-fno-gpu-flush-denormals-to-zero", "-fno-fast-math", "-ffp-contract=on",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-fconstexpr-steps=200000000", "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Wall", "-I", os.path.join(ROOT, "include"),
]


NATIVE_OUT = os.path.join(HERE, "_native.so")
NATIVE_SOURCE = os.path.join(CSRC, "binding.cpp")
CXX = os.environ.get("CXX", "g++")


def build(verbose: bool = False, extra=()) -> str:
    _compile([HIPCC, *FLAGS, *extra, "-o", OUT + ".tmp", *SOURCES], OUT, verbose)
    if _torch_headers():
        build_native(verbose)        # links libfewbit.so, so after it
    else:
        print("no torch with headers here: _native.so is not built, the Python package needs it")
    return OUT


def _torch_headers() -> bool:
    try:
        import torch
    except ImportError:
        return False
    return os.path.isdir(os.path.join(os.path.dirname(torch.__file__), "include", "torch", "csrc"))


def build_native(verbose: bool = False) -> str:
    import sysconfig
    import torch
    from torch.utils.cpp_extension import include_paths
    libs = os.path.join(os.path.dirname(torch.__file__), "lib")
    rocm = os.path.dirname(os.path.dirname(HIPCC))
    includes = [os.path.join(ROOT, "include"), *include_paths(), os.path.join(rocm, "include"),
                sysconfig.get_paths()["include"]]
    _compile([CXX, "-std=c++17", "-O2", "-fPIC", "-shared", "-Wall",
              # the HIP headers ask for the platform where hipcc does not compile
              "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
              f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
              *(f"-I{d}" for d in includes), "-o", NATIVE_OUT + ".tmp", NATIVE_SOURCE,
              f"-L{HERE}", "-lfewbit", f"-L{libs}", "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_hip",
              "-ltorch_python", "-Wl,-rpath,$ORIGIN"], NATIVE_OUT, verbose)
    return NATIVE_OUT


def _compile(cmd, out: str, verbose: bool) -> None:
    tmp = out + ".tmp"
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass does not know the packed-fp32 target feature: harmless
    msgs = [ln for ln in (r.stdout + r.stderr).splitlines()
            if "packed-fp32-ops" not in ln and ln.strip()]
    if r.returncode != 0:
        raise RuntimeError(f"{os.path.basename(cmd[0])} failed:\n" + "\n".join(msgs))
    if verbose and msgs:
        print("\n".join(msgs))
    os.replace(tmp, out)


if __name__ == "__main__":
    print(build(verbose=True))
