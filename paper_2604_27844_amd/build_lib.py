"""Build libzipccl.so (the codec) and libzipccl_yardstick.so (the benchmark's plain-copy kernel) in-tree with
hipcc for gfx950 (cross-compiles without a GPU), and the module zipccl_python (the binding's calls) with the host compiler."""
import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libzipccl.so")
YARDSTICK = os.path.join(HERE, "libzipccl_yardstick.so")
SOURCES = ["zipccl_compress.hip", "zipccl_decompress.hip", "zipccl_aux.hip", "zipccl_host.cpp"]
HEADERS = [os.path.join(CSRC, "zipccl_internal.h"), os.path.join(CSRC, "zipccl_device.h"),
           os.path.join(ROOT, "include", "zipccl.h")]
TARGETS = {LIB: [os.path.join(CSRC, s) for s in SOURCES],
           YARDSTICK: [os.path.join(CSRC, "zipccl_yardstick.hip")]}


def python_module():
    """The module's file.  Compiled in are this interpreter's object layouts and this torch's tensor layout, so both are in its
    name: what was built for others is not found."""
    import torch
    return os.path.join(HERE, f"zipccl_python-torch{torch.__version__}{sysconfig.get_config_var('EXT_SUFFIX')}")


def _sources(target):
    return TARGETS.get(target) or [os.path.join(CSRC, "zipccl_python.cpp")]


def stale(lib=LIB):
    if not os.path.exists(lib):
        return True
    t = os.path.getmtime(lib)
    deps = _sources(lib) + HEADERS + [os.path.join(ROOT, "include", "zipccl_yardstick.h")]
    return any(os.path.getmtime(d) > t for d in deps)


def _python_command(sources, out):
    import torch
    from torch.utils import cpp_extension
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
           "-I", os.path.join(ROOT, "include")]
    for path in cpp_extension.include_paths() + [sysconfig.get_paths()["include"]]:
        cmd += ["-isystem", path]
    cmd += sources + ["-o", out, "-L", HERE, "-lzipccl", "-Wl,-rpath,$ORIGIN"]
    for path in cpp_extension.library_paths():
        cmd += ["-L", path]
    return cmd + ["-lc10", "-ltorch_cpu", "-ltorch", "-ltorch_python"]


def hip_command(sources, out, flags=()):
    return [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-Wall", "-Wno-unused-command-line-argument",
            "-I", os.path.join(ROOT, "include"), "-I", CSRC, *flags, *sources, "-o", out]


def build(force=True, verbose=False, lib=None):
    """Compile every target (or the one named); returns the codec library's path.  Without torch the module, which only
    takes its tensors, is left out."""
    targets = [*TARGETS] if lib is None else [lib]
    if lib is None:
        try:
            targets.append(python_module())
        except ImportError:
            pass
    for target in targets:
        if not force and not stale(target):
            continue
        sources = _sources(target)
        tmp = target + f".{os.getpid()}.tmp"
        cmd = hip_command(sources, tmp) if target in TARGETS else _python_command(sources, tmp)
        if verbose:
            print(" ".join(cmd))
        subprocess.check_call(cmd)
        os.replace(tmp, target)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
