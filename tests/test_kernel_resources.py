"""What the compiler made of the kernels (arxiv 2411.01238, Section 3.1: the products are bound by their inner loops): no
register of theirs lies in scratch memory.  A reload between an epilogue's stores waits for every store before it, and one in
a loader holds up a slice; neither changes a result, so no other test sees it."""
import os
import re
import struct
import subprocess

import pytest

from paper_2411_01238_amd import sdrop

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"

# Mangled name -> bytes of scratch memory that these may use, with the reason.
ALLOWED = [
    # the pair list's 16-bit form holds two epilogues (rows and transposed): one or two registers, outside its loops
    (r"gemm_persistent_dx_kernelI.*Li128ELi256ELi2ELi2ELi0ELb0ELb1ELb0E|bwd_fused_kernelI.*Li256ELb1ELb0ELi(128|256)E", 16),
    # eq. (1) under a gate on 128 x 256 tiles: gate values beside 128 accumulators, 16-bit results only
    (r"gemm_persistent_kernelILi0E.*DF16[b_]Li128ELi256ELi1ELi4ELi[25]ELb0E", 128),
    # eq. (2) with a ragged reduction, a workgroup per tile: a local array that is indexed, no spill
    (r"gemm_kernelILi1E.*Li128ELi128ELi2ELi2ELb1ELb0ELb[01]E", 64),
]


def _kernels(path):
    """(name, scratch bytes, spilled vector registers) of every gfx950 kernel embedded in a library."""
    data = open(path, "rb").read()
    out = []
    for m in re.finditer(re.escape(MAGIC), data):
        p = m.start() + len(MAGIC)
        (n,) = struct.unpack_from("<Q", data, p)
        p += 8
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, p)
            target = data[p + 24:p + 24 + length].decode()
            p += 24 + length
            if "gfx950" not in target or not size:
                continue
            obj = data[m.start() + off:m.start() + off + size]
            r = subprocess.run([READELF, "--notes", "-"], input=obj, stdout=subprocess.PIPE, check=True)
            for block in re.split(r"\n  - \.agpr_count", r.stdout.decode())[1:]:
                field = {k: int(re.search(r"\.%s:\s+(\d+)" % k, block)[1]) for k in ("private_segment_fixed_size", "vgpr_spill_count")}
                out.append((re.findall(r"\.name:\s+(_Z\S+)", block)[-1], field["private_segment_fixed_size"], field["vgpr_spill_count"]))
    return out


@pytest.mark.skipif(not os.path.exists(READELF), reason="needs the toolchain's readelf")
def test_no_kernel_keeps_registers_in_scratch_memory():
    kernels = _kernels(sdrop.LIB_PATH)
    assert len(kernels) > 100                       # (the bundles were found and read)
    bad = []
    for name, scratch, spills in kernels:
        allowed = max([b for pattern, b in ALLOWED if re.search(pattern, name)], default=0)
        if scratch > allowed:
            bad.append((name, scratch, spills))
    assert not bad, "%d kernels with scratch memory: %s" % (len(bad), bad[:5])
