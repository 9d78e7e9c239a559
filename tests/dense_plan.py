"""Which kernel and tile a dense convolution takes, asked of the library's own rule without a GPU."""
import ctypes
import functools
import os
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2109_00170_amd", "csrc")
KINDS = ("gather", "float32", "split")


@functools.lru_cache(None)
def _library():
    with tempfile.TemporaryDirectory() as d:
        so = os.path.join(d, "dense_plan.so")
        subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC,
                               os.path.join(HERE, "native", "dense_plan.cpp"), "-o", so])
        return ctypes.CDLL(so)


def dense_plan(k, stride, Cin, Cout, H, W, N, cus=256, few=True):
    """(kernel size, "gather" / "float32" / "split", channels, pixels, positions per thread) of the tile, and its positions
    and LDS bytes; (kernel size, "few", 32, 32, 0) where the launch is left to the kernel of small launches
    (few=False: the tile it would take otherwise)."""
    out = (ctypes.c_int * 8)()
    _library().dense_plan((ctypes.c_int * 7)(N, Cin, Cout, H, W, k, stride), cus, out)
    if few and out[7]:
        return (k, "few", 32, 32, 0), 0, 64 * 1024
    return (k, KINDS[out[0]]) + tuple(out[1:4]), out[4], out[6]
