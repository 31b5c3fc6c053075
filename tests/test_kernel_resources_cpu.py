"""Registers of the built half-pass kernels, the ablation build's among them, from the metadata the compiler leaves in the
library: 4 waves on a SIMD and nothing in scratch memory."""
import os
import re
import shutil
import struct
import subprocess

import pytest

READELF = next((p for p in ("/opt/rocm/llvm/bin/llvm-readelf", shutil.which("llvm-readelf")) if p and os.path.exists(p)),
               None)


def code_objects(lib):
    """The gfx950 code objects of the library's offload bundles."""
    data = open(lib, "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        n, pos = struct.unpack_from("<Q", data, at + len(magic))[0], at + len(magic) + 8
        for _ in range(n if n < 16 else 0):
            off, size, length = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + length]
            pos += 24 + length
            if b"gfx950" in name and size:
                yield data[at + off:at + off + size]
        at = data.find(magic, at + 1)


@pytest.mark.skipif(READELF is None, reason="needs llvm-readelf")
def test_half_pass_kernels_spill_nothing(tmp_path):
    import paper_1805_07920_amd as amh

    if not os.path.exists(amh.LIB_PATH):
        from paper_1805_07920_amd import build

        build.build()
    kernels = {}
    for i, obj in enumerate(code_objects(amh.LIB_PATH)):
        f = tmp_path / f"{i}.elf"
        f.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(f)], capture_output=True, text=True, check=True).stdout
        for part in notes.split("- .agpr_count:")[1:]:
            field = lambda k: re.search(rf"\.{k}:\s*(\S+)", part).group(1)
            kernels[field("symbol")] = [int(field(k)) for k in ("private_segment_fixed_size", "vgpr_spill_count",
                                                                "vgpr_count")]
    half = {k: v for k, v in kernels.items() if re.search(r"(pass|batch|persist|ablation)_kernelILi", k)}
    # float32 and float16 sources x tile rows 1 .. 4, few views 1 and 4, batches 2 .. 4, and twice 2 and 4
    assert len(half) == 8 + 4 + 6 + 4 + 4
    for name, (scratch, spilled, vgprs) in sorted(half.items()):
        assert scratch == 0 and spilled == 0 and vgprs <= 128, (name, scratch, spilled, vgprs)
