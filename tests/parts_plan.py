"""How the kernels that walk chunks share their groups out, asked of the library's own rule without a GPU."""
import ctypes
import functools
import os
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2109_00170_amd", "csrc")


@functools.lru_cache(None)
def _library():
    with tempfile.TemporaryDirectory() as d:
        so = os.path.join(d, "parts_plan.so")
        subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC,
                               os.path.join(HERE, "native", "parts_plan.cpp"), "-o", so])
        return ctypes.CDLL(so)


def parts_plan(V, G, npt, ngt, cols, nchunks=1, nw=16, gpt=None, three=True, alone=False, wide=False, strided=False,
               stride2=False, uneven=False, unaligned=False, shared=False, cus=256):
    """(group tiles, groups of one, wavefronts that share a group), or None where the launch keeps several groups per
    wavefront.  `cols`: kept columns of a group, in the mean."""
    out = (ctypes.c_int * 3)()
    gpt = -(-G // ngt) if gpt is None else gpt
    _library().parts_plan((ctypes.c_int * 15)(cus, nw, V, G, npt, ngt, gpt, three, alone, wide, strided, stride2, uneven,
                                              unaligned, shared),
                          (ctypes.c_float * 2)(cols / nchunks, cols), out)
    return tuple(out) if out[0] else None


def groups_of_tile(G, ngt, npt, nw, ug, slots):
    return _library().groups_of_tile(G, ngt, npt, nw, ug, slots)
