"""What the compiler reports about the built kernels: registers moved to scratch memory cost every
workgroup a trip to memory, and nothing else shows them.  In k_client_step the compiler has put those
moves into a branch of one lane, so that the others read back what they had never stored: candidates of
other tensors, then, in lists longer than LDS holds."""
import os
import re
import shutil
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1805_08768_amd", "libsbc.so")
READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _spills(tmp_path):
    """{kernel symbol: vector registers spilled} from the metadata of the library's gfx950 code object."""
    data = open(LIB, "rb").read()
    start = data.index(MAGIC)
    at = start + len(MAGIC)
    (count,) = struct.unpack_from("<Q", data, at)
    at += 8
    for _ in range(count):
        off, size, id_len = struct.unpack_from("<QQQ", data, at)
        name = data[at + 24:at + 24 + id_len].decode()
        at += 24 + id_len
        if "gfx950" in name:
            path = tmp_path / "code.o"
            path.write_bytes(data[start + off:start + off + size])
            notes = subprocess.run([READELF, "--notes", str(path)], check=True, capture_output=True, text=True).stdout
            return {m.group(1): int(m.group(2))
                    for m in re.finditer(r"\.symbol:\s+(\S+)\.kd.*?\.vgpr_spill_count:\s+(\d+)", notes, re.S)}
    raise AssertionError("no gfx950 code object in the library")


@pytest.mark.skipif(not os.path.exists(LIB) or not os.path.exists(READELF), reason="library not built here")
def test_kernels_keep_their_registers(tmp_path):
    spills = _spills(tmp_path)
    for kernel in ("k_accumulate_filter", "k_client_step", "k_threshold", "k_apply", "k_emit", "k_finish_message", "k_decode", "k_average_apply"):
        found = {s: n for s, n in spills.items() if kernel in s}
        assert found and not any(found.values()), found
