"""Resources the compiler gave the kernels of the built library (the metadata of its gfx950 code objects): the kernels named here keep
everything in registers.  A spilled register costs them 10 to 50 % (measured on conv_kernel behind a linked depthwise producer with a
global average, and on fire_kernel), and nothing else shows it: results are the same."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2302_00282_amd import xenos as X

READELF = next((p for p in (shutil.which("llvm-readelf"), "/opt/rocm/llvm/bin/llvm-readelf") if p and os.path.exists(p)), None)
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(data):
    """The gfx950 ELF images of the offload bundles in a shared library."""
    at = data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + len(MAGIC))
        pos = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, tlen = struct.unpack_from("<QQQ", data, pos)
            triple = data[pos + 24:pos + 24 + tlen].decode()
            pos += 24 + tlen
            if "gfx950" in triple and size:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, pos)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if READELF is None:
        pytest.skip("no llvm-readelf")
    out = {}
    with open(X.LIB_PATH, "rb") as f:
        images = list(_code_objects(f.read()))
    for i, image in enumerate(images):
        path = tmp_path_factory.mktemp("co") / f"{i}.co"
        path.write_bytes(image)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for block in re.split(r"\n\s+- \.agpr_count", notes)[1:]:
            field = lambda k: re.search(r"\." + k + r":\s+(\S+)", block).group(1)
            out[field("name")] = (int(field("vgpr_spill_count")), int(field("private_segment_fixed_size")))
    assert out
    return out


@pytest.mark.parametrize("kernel", ["conv_kernel", "fire_kernel", "dwpw_kernel", "pwdw_kernel", "unit_kernel", "dw_kernel", "splitk_finish_kernel", "fc_stream_kernel"])
def test_no_vector_register_is_spilled(kernels, kernel):
    found = {k: v for k, v in kernels.items() if re.search(r"\d" + kernel + r"I|\d" + kernel + r"E", k)}
    assert found, kernel
    assert not {k: v for k, v in found.items() if v != (0, 0)}
