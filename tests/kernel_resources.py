"""Registers and LDS of the kernels in the built library, from the metadata of
the gfx950 code objects that the build put into it."""

import os
import re
import struct
import subprocess
import tempfile

from paper_2609_00993_amd import moepd

READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
VGPRS_PER_LANE = 512  # of a SIMD, shared by its waves
VGPR_UNIT = 8
LDS_UNITS = 128  # of a CU, 1280 bytes each


def lds_units(nbytes):
    return -(-nbytes // 1280)


def _code_objects():
    data = open(moepd.LIB_PATH, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            ident = data[p + 24:p + 24 + idlen]
            p += 24 + idlen
            if b"gfx950" in ident and size:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + 1)


def kernels():
    """{demangled kernel name: (VGPRs with AGPRs as allocated, LDS bytes)}."""
    got = {}
    for elf in _code_objects():
        with tempfile.NamedTemporaryFile(suffix=".co") as f:
            f.write(elf)
            f.flush()
            notes = subprocess.run([READELF, "--notes", f.name], stdout=subprocess.PIPE, text=True, check=True).stdout
        for block in re.split(r"\n  - \.agpr_count:", notes)[1:]:
            name = re.search(r"\.name: +(\S+)", block).group(1)
            vgprs = int(re.search(r"\.vgpr_count: +(\d+)", block).group(1))
            lds = int(re.search(r"\.group_segment_fixed_size: +(\d+)", block).group(1))
            got[name] = (-(-vgprs // VGPR_UNIT) * VGPR_UNIT, lds)
    names = subprocess.run(["c++filt"], input="\n".join(got), stdout=subprocess.PIPE, text=True, check=True).stdout
    return dict(zip((n.split("(")[0].replace("moepd::", "").replace("void ", "") for n in names.split("\n")),
                    got.values()))
