"""The one-step sweeps, solo and batched, of the 4- and 2-byte storages keep
their values in vector registers: a sweep compiled for more wavefronts than its
registers allow spills kilobytes a lane and takes many times as long, without a
wrong result.  Read from the kernels' metadata in the built library."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_1710_02065_amd import build

READELF = os.path.join(os.path.dirname(build.HIPCC), "..", "llvm", "bin", "llvm-readelf")


def code_objects(data):
    """Device code objects in the library's offload bundles."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(count):
            offset, size, n = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + n].decode()
            p += 24 + n
            if build.ARCH in name and size:
                yield data[at + offset:at + offset + size]
        at = data.find(magic, at + 24)


def test_sweeps_spill_no_vector_register(tmp_path):
    if not os.path.exists(build.LIB) or not shutil.which(READELF):
        pytest.skip("library or llvm-readelf missing")
    with open(build.LIB, "rb") as f:
        data = f.read()
    seen, bad = 0, []
    for k, code in enumerate(code_objects(data)):
        path = tmp_path / ("%d.co" % k)
        path.write_bytes(code)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True,
                               check=True).stdout
        for entry in notes.split("- .agpr_count")[1:]:
            name = re.search(r"\.name:\s+(\S+)", entry).group(1)
            if re.search(r"(7k_sweep|7k_batch)I.*Store(F32|F32S|F16S)E", name):
                seen += 1
                if int(re.search(r"\.vgpr_spill_count:\s+(\d+)", entry).group(1)):
                    bad.append(name)
    # 9 lattices, orders and collisions, 3 storages; 4 solo sweeps, 2 batched ones
    assert seen == 9 * 3 * 6 and not bad, (seen, bad)
