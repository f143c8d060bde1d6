"""Register use of the attention kernels, read from the metadata of the library
that was built here.  No kernel spills vector registers, and those of the padded
caches (attn_main's fifth template argument is false) no scalar ones either: a
scalar register spilled to a vector lane is read back in the tile loop, and nine
such reads per tile cost 2% of a call."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2606_18394_amd import build

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(path):
    """The gfx950 code objects of a library's offload bundles."""
    data = open(path, "rb").read()
    at = data.find(BUNDLE)
    while at >= 0:
        count, = struct.unpack_from("<Q", data, at + len(BUNDLE))
        pos = at + len(BUNDLE) + 8
        for _ in range(count):
            offset, size, n = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + n]
            pos += 24 + n
            if b"gfx950" in name:
                yield data[at + offset:at + offset + size]
        at = data.find(BUNDLE, at + 1)


@pytest.mark.skipif(not shutil.which(READELF), reason="needs llvm-readelf")
def test_attention_kernels_do_not_spill(tmp_path):
    if not os.path.exists(build.LIB):
        build.build()
    seen = 0
    for k, obj in enumerate(code_objects(build.LIB)):
        elf = tmp_path / f"{k}.o"
        elf.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(elf)], capture_output=True, text=True,
                               check=True).stdout
        for entry in re.split(r"\n\s*- \.agpr_count:", notes)[1:]:
            name = re.search(r"\n\s*\.name:\s*(\S+)", entry).group(1)
            if "attn_main" not in name and "attn_packed" not in name:
                continue
            seen += 1
            paged = re.search(r"attn_mainI(?:Li\d+E){4}Lb1E", name)
            fields = [".vgpr_spill_count", ".private_segment_fixed_size"]
            for field in fields + ([] if paged else [".sgpr_spill_count"]):
                assert re.search(rf"\n\s*\{field}:\s*0\n", entry), (name, field)
    assert seen >= 20
