"""Build libattncache.so (HIP, gfx950 only) and the binding's tensor check in-tree next to the sources."""
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libattncache.so")
SOURCES = ["api.hip", "apply.hip", "exact.hip", "insert.hip", "project.hip", "search.hip"]
HEADERS = ["common.hpp", "f32_tile.hpp", "launch.hpp", "row_stream.hpp", "short_tile.hpp", "split_tile.hpp", os.path.join("..", "..", "include", "attncache.h")]
ARG = os.path.join(HERE, "_tensor_arg.so")
ARG_SOURCE = "tensor_arg.cpp"

# -packed-fp32-ops is switched off: the compiler must not form packed fp32 instructions
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-fno-gpu-rdc",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall",
         "-Wno-unused-command-line-argument", "-Wl,-z,defs"]


def _older(out, sources) -> bool:
    return not os.path.exists(out) or any(os.path.getmtime(os.path.join(CSRC, f)) > os.path.getmtime(out) for f in sources)


def stale() -> bool:
    return _older(LIB, SOURCES + HEADERS) or _older(ARG, [ARG_SOURCE])


def _lib_command():
    return ["hipcc"] + FLAGS + [os.path.join(CSRC, f) for f in SOURCES] + ["-o", LIB]


def _arg_command():
    import torch
    from torch.utils.cpp_extension import include_paths
    torch_lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    return (["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
             f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"] +
            [f"-I{p}" for p in include_paths() + [sysconfig.get_path("include")]] +
            [os.path.join(CSRC, ARG_SOURCE), f"-L{torch_lib}", "-ltorch_python", "-ltorch_cpu", "-lc10", "-o", ARG])


def _build_arg(verbose: bool) -> None:
    """The tensor check needs torch's headers, Python's and g++; the library needs none of them, and the binding does
    without the check (slower), so a machine that lacks one is told so and gets the library all the same."""
    try:
        cmd = _arg_command()
        if verbose:
            print(" ".join(cmd))
        subprocess.run(cmd, check=True)
    except (ImportError, OSError, subprocess.CalledProcessError) as e:
        if os.path.exists(ARG):   # one of other sources
            os.remove(ARG)
        print(f"{os.path.basename(ARG)} is not built ({e}): tensor arguments are checked in Python", file=sys.stderr)


def build(force: bool = True, verbose: bool = False) -> str:
    lib = None
    if force or _older(LIB, SOURCES + HEADERS):
        cmd = _lib_command()
        if verbose:
            print(" ".join(cmd))
        lib = subprocess.Popen(cmd)
    try:
        if force or _older(ARG, [ARG_SOURCE]):
            _build_arg(verbose)
    finally:
        code = lib.wait() if lib else 0
    if code:
        raise subprocess.CalledProcessError(code, cmd)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose=True))
