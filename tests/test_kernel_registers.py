"""The built kernels keep their state in registers: none has a private segment (scratch memory) but the K product's form
of five waves per SIMD, which holds up to ten registers there and gains more from the fifth wave."""
import os
import re
import struct
import subprocess

import pytest

from paper_2512_24449_amd import binding

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def _code_objects(lib):
    """The gfx950 code objects of the offload bundles in a shared library."""
    data, magic, pos = open(lib, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (pos := data.find(magic, pos)) >= 0:
        at = pos + 32
        for _ in range(struct.unpack_from("<Q", data, pos + 24)[0]):
            offset, size, n = struct.unpack_from("<QQQ", data, at)
            if b"gfx950" in data[at + 24:at + 24 + n]:
                yield data[pos + offset:pos + offset + size]
            at += 24 + n
        pos += len(magic)


def test_no_kernel_spills_vector_registers(tmp_path):
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    binding.lib()
    scratch = {}
    for i, code in enumerate(_code_objects(binding.library_path())):
        path = tmp_path / ("%d.co" % i)
        path.write_bytes(code)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for kernel in re.split(r"\n\s+- \.agpr_count", notes)[1:]:
            name = re.findall(r"\.name:\s+(_Z\S+)", kernel)[-1]
            scratch[name] = int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", kernel)[1])
    assert len(scratch) > 50, "the kernels' metadata was not found"
    assert not {k: n for k, n in scratch.items() if n > (48 if "k_planes_kernel" in k else 0)}
