"""tests/impatient/libzipccl_impatient.so: a copy of the compress side whose workgroups do not wait for one another's counts, for
the tests of what they do instead (test_gpu_chain.py)."""
import os
import subprocess

from paper_2604_27844_amd import build_lib

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "impatient")
LIB = os.path.join(HERE, "libzipccl_impatient.so")


def build():
    sources = [os.path.join(build_lib.CSRC, "zipccl_compress.hip"), os.path.join(build_lib.CSRC, "zipccl_host.cpp"), os.path.join(HERE, "rest.cpp")]
    tmp = LIB + f".{os.getpid()}.tmp"
    subprocess.check_call(build_lib.hip_command(sources, tmp, ["-DZIPCCL_CHAIN_PATIENCE=0", "-Wl,-Bsymbolic"]))
    os.replace(tmp, LIB)
    return LIB
