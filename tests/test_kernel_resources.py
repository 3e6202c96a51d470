"""Registers and scratch memory of the streaming kernel, as the compiler recorded them in the built library."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2601_23180_amd.binding import LIB_PATH

READELF = shutil.which("llvm-readelf", path="/opt/rocm/llvm/bin:" + os.environ.get("PATH", ""))
pytestmark = pytest.mark.skipif(READELF is None, reason="no llvm-readelf")


def kernels(tmp_path):
    """Metadata of every kernel of the library's gfx950 code objects: symbol -> {field: value}."""
    blob, found, at = open(LIB_PATH, "rb").read(), {}, 0
    while (at := blob.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        entry = at + 32
        for _ in range(struct.unpack_from("<Q", blob, at + 24)[0]):
            offset, size, name = struct.unpack_from("<QQQ", blob, entry)
            if size and b"gfx950" in blob[entry + 24:entry + 24 + name]:
                part = tmp_path / "code_object"
                part.write_bytes(blob[at + offset:at + offset + size])
                notes = subprocess.run([READELF, "--notes", str(part)], capture_output=True, text=True, check=True).stdout
                for text in notes.split("- .agpr_count:")[1:]:
                    fields = dict(re.findall(r"\.(\w+):\s+(\S+)", text))
                    found[fields["symbol"]] = fields
            entry += 24 + name
        at += 24
    return found


def test_streaming_kernels_keep_to_their_registers(tmp_path):
    """No scratch memory and no register spilt, whether one workgroup finishes a tile or all of them do."""
    seen = {0: 0, 1: 0}
    for symbol, k in kernels(tmp_path).items():
        m = re.match(r"_ZN2ts13k_gemm_streamI(?:Li\d+E){5}(?:Lb([01])E)?E", symbol)
        if not m:
            continue
        seen[int(m[1] or 0)] += 1
        assert int(k["private_segment_fixed_size"]) == 0, symbol
        assert int(k["vgpr_spill_count"]) == 0 and int(k["sgpr_spill_count"]) == 0, symbol
    assert seen[0] > 100 and seen[1] > 30
