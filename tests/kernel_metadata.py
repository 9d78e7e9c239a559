"""Registers and memory of the library's kernels, as the compiler recorded them in the code objects of libalcs.so."""
import collections
import functools
import os
import re
import struct
import subprocess
import tempfile

import paper_2109_00170_amd as alcs

Kernel = collections.namedtuple("Kernel", "vgprs sgpr_spills vgpr_spills scratch lds")
LLVM = "/opt/rocm/llvm/bin"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@functools.lru_cache(None)
def kernels():
    """{demangled name without arguments: Kernel}"""
    out = {}
    with tempfile.TemporaryDirectory() as d:
        section = os.path.join(d, "fatbin")
        subprocess.check_call(["objcopy", "-O", "binary", "--only-section=.hip_fatbin", alcs.library_path(), section])
        with open(section, "rb") as f:
            data = f.read()
        at = data.find(MAGIC)
        while at >= 0:
            entry = at + 32
            for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
                offset, size, length = struct.unpack_from("<QQQ", data, entry)
                target = data[entry + 24:entry + 24 + length].decode()
                entry += 24 + length
                if "gfx950" not in target or not size:
                    continue
                path = os.path.join(d, "object")
                with open(path, "wb") as f:
                    f.write(data[at + offset:at + offset + size])
                notes = subprocess.check_output([os.path.join(LLVM, "llvm-readelf"), "--notes", path], text=True)
                for k in re.split(r"\n\s+- \.agpr_count", notes)[1:]:
                    def field(name):
                        return int(re.search(r"\.%s:\s+(\d+)" % name, k)[1])
                    out[re.search(r"\.name:\s+(\S+)", k)[1]] = Kernel(
                        field("vgpr_count"), field("sgpr_spill_count"), field("vgpr_spill_count"),
                        field("private_segment_fixed_size"), field("group_segment_fixed_size"))
            at = data.find(MAGIC, at + len(MAGIC))
    plain = subprocess.run(["c++filt"], input="\n".join(out), text=True, check=True,
                           stdout=subprocess.PIPE).stdout.split("\n")
    return {re.sub(r"^void ", "", p).split("(alcs")[0]: k for p, k in zip(plain, out.values())}
