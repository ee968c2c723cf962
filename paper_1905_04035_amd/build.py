"""Compiles csrc/*.hip for gfx950 into libts_densify.so next to this file, and csrc/marshal.cpp, the binding's
marshalling (host code against PyTorch's headers), into the extension module _marshal."""
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SRCS = [os.path.join(HERE, "csrc", f) for f in ("ts_densify.hip", "ts_accumulate.hip")]
LIB = os.path.join(HERE, "libts_densify.so")
LIB_SAN = os.path.join(HERE, "libts_densify_san.so")     # host code under ASan + UBSan (checks of the host logic)
INCLUDE = os.path.join(ROOT, "include")

MARSHAL_SRC = os.path.join(HERE, "csrc", "marshal.cpp")
MARSHAL_USES = [MARSHAL_SRC, os.path.join(INCLUDE, "ts_densify.h")]
MARSHAL = os.path.join(HERE, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))     # of this interpreter

MARSHAL_SAN = os.path.join(HERE, "_marshal_san" + sysconfig.get_config_var("EXT_SUFFIX"))

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # keep the compiler from forming packed-fp32 instructions out of float4 arithmetic
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wextra", "-I", INCLUDE,
]


SAN_FLAGS = ["-g", "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
             "-Xarch_host", "-fno-sanitize-recover=undefined", "-shared-libsan"]
CLANGXX = os.environ.get("CLANGXX", "/opt/rocm/llvm/bin/clang++")
MARSHAL_SAN_FLAGS = ["-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-shared-libsan"]


def marshal_command(sanitize: bool = False):
    import torch

    root = os.path.dirname(torch.__file__)
    return [CLANGXX if sanitize else os.environ.get("CXX", "g++"), *(MARSHAL_SAN_FLAGS if sanitize else []), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wextra",
            "-Wno-missing-field-initializers", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            "-isystem", os.path.join(root, "include"), "-isystem", sysconfig.get_paths()["include"], "-I", INCLUDE,
            "-o", MARSHAL_SAN if sanitize else MARSHAL, MARSHAL_SRC, "-L", os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]


def build_marshal(force: bool = True, sanitize: bool = False) -> str:
    """force=False: only if it is missing or older than what it is made from (it calls the library's entry points by
    their addresses, with the signatures of the header that it was compiled with)."""
    module = MARSHAL_SAN if sanitize else MARSHAL
    old = not os.path.exists(module) or os.path.getmtime(module) < max(os.path.getmtime(f) for f in MARSHAL_USES)
    if force or old:
        cmd = marshal_command(sanitize)
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError(cmd[0] + " failed:\n" + res.stderr)
    return module


def build(force: bool = True, verbose: bool = False, sanitize: bool = False) -> str:
    """sanitize=True: a second library whose HOST code runs under the address and
    undefined-behaviour sanitizers (device code unchanged), and a second module that does; the loading
    process must have clang's shared sanitizer runtime preloaded."""
    lib = LIB_SAN if sanitize else LIB
    if force or not os.path.exists(lib):
        build_library(lib, verbose, sanitize)
    build_marshal(force, sanitize)
    return lib


def build_library(lib: str, verbose: bool = False, sanitize: bool = False) -> None:
    cmd = [HIPCC] + FLAGS + (SAN_FLAGS if sanitize else []) + ["-o", lib] + SRCS
    if verbose:
        print(" ".join(cmd))
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + err)
    if err.strip() and verbose:
        print(err)


if __name__ == "__main__":
    print(build(force=True, verbose=True, sanitize="--sanitize" in sys.argv))
    sys.exit(0)
