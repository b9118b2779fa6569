"""Headers of the library that are plain C++, compiled for the host."""
import ctypes as C
import functools
import os
import subprocess
import tempfile

from paper_2408_12525_amd import workloads as wl

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2408_12525_amd", "csrc")


@functools.lru_cache(None)
def library(source):
    """The C++ text `source`, which includes headers of csrc/, as a loaded library."""
    with tempfile.TemporaryDirectory() as d:
        with open(os.path.join(d, "rule.cpp"), "w") as f:
            f.write(source)
        so = os.path.join(d, "rule.so")
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-shared", "-fPIC", "-I", CSRC, f.name, "-o", so], check=True)
        return C.CDLL(so)


def call(source, numbers, n_out):
    """What its function `rule(const int64_t* in, int64_t* out)` gives for these numbers."""
    v, out = (C.c_int64 * len(numbers))(*[int(n) for n in numbers]), (C.c_int64 * n_out)()
    library(source).rule(v, out)
    return tuple(out)


def obs_stride(cfg):
    """Bytes from one level's observation to the next: what pcgrl_create works out."""
    one, pitch = wl.obs_bytes(cfg), cfg.get("obs_pitch", 0)
    return -(-one // 128) * 128 if pitch < 0 else pitch if pitch > 0 else one
