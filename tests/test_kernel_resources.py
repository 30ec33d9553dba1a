"""Registers of the built kernels, from the code objects' metadata: the limits
that their occupancy rests on (512 vector registers per SIMD lane: 128 each for
four waves, 168 for three) and no spilled register where none is expected."""
import os
import re
import struct
import subprocess

import pytest

sf = pytest.importorskip("paper_1512_02951_amd")

TOOLS = "/opt/rocm/llvm/bin"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled name: (vector registers, scratch bytes)} of every kernel."""
    objcopy, readelf = (os.path.join(TOOLS, t) for t in ("llvm-objcopy", "llvm-readelf"))
    if not (os.path.exists(sf.LIB_PATH) and os.path.exists(objcopy) and os.path.exists(readelf)):
        pytest.skip("library or LLVM tools missing")
    d = tmp_path_factory.mktemp("code")
    fat = str(d / "fat.bin")
    subprocess.run([objcopy, "--dump-section=.hip_fatbin=" + fat, sf.LIB_PATH, str(d / "host.so")], check=True)
    data = open(fat, "rb").read()
    out = {}
    at = data.find(MAGIC)
    while at >= 0:
        p = at + len(MAGIC)
        (n,) = struct.unpack_from("<Q", data, p)
        p += 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            ident = data[p + 24:p + 24 + idlen].decode()
            p += 24 + idlen
            if "gfx950" not in ident:
                continue
            co = d / "code.co"
            co.write_bytes(data[at + off:at + off + size])
            notes = subprocess.run([readelf, "--notes", str(co)], check=True, capture_output=True, text=True).stdout
            for k in notes.split("- .agpr_count")[1:]:
                name = re.search(r"\.name:\s+(_Z\S+)", k).group(1)
                out[name] = (int(re.search(r"\.vgpr_count:\s+(\d+)", k).group(1)),
                             int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", k).group(1)))
        at = data.find(MAGIC, at + 1)
    return out


# kernels in which four waves share a SIMD, and (strong frag) three
@pytest.mark.parametrize("name,count,limit", [("pixel_frag_kernelILi%d+ELb0E", 4, 128),
                                              ("pixel_frag_kernelILi%d+ELb1E", 4, 168), ("pixel_defrag_kernel", 8, 128),
                                              ("dwt_frag_kernel", 1, 128), ("dwt_defrag_kernel", 1, 128),
                                              ("lp_frag_kernel", 10, 128), ("lp_defrag_kernel", 10, 128)])
def test_registers_leave_room_for_the_waves(kernels, name, count, limit):
    found = {k: v for k, v in kernels.items() if re.search(r"\d" + name.replace("%d", r"\d"), k)}
    assert len(found) == count, sorted(kernels)
    for k, (vgprs, scratch) in found.items():
        assert vgprs <= limit and scratch == 0, (k, vgprs, scratch)
