"""No kernel of the built library uses scratch memory: a reload inside a loop that keeps direct-to-LDS loads in flight waits for all of them (the
input gradient at block size 128 took 857 us with two reloads a stage, 698 without).  Reads the kernel descriptors of this repository's own build."""
import os
import re
import struct
import subprocess

from paper_2403_12422_amd import build

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")


def code_objects(data):
    """The gfx950 code objects of the bundles, one for each source."""
    at = data.find(MAGIC)
    while at >= 0:
        pos = at + len(MAGIC)
        (count,) = struct.unpack_from("<Q", data, pos)
        pos += 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, pos)
            target = data[pos + 24:pos + 24 + length]
            pos += 24 + length
            if b"gfx950" in target:
                yield data[at + offset:at + offset + size]
        at = data.find(MAGIC, at + len(MAGIC))


def test_no_scratch_memory(tmp_path):
    with open(build.LIB, "rb") as f:
        objects = list(code_objects(f.read()))
    assert len(objects) == len(build.sources()) - 2      # jf_api.hip and jf_linear.hip have no kernels
    kernels, spilled = 0, []
    for i, blob in enumerate(objects):
        path = tmp_path / f"{i}.co"
        path.write_bytes(blob)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True, timeout=60).stdout
        sizes = [int(n) for n in re.findall(r"\.private_segment_fixed_size:\s+(\d+)", notes)]
        names = re.findall(r"\.symbol:\s+(\S+)", notes)
        assert len(sizes) == len(names) > 0
        kernels += len(names)
        spilled += [(n, s) for n, s in zip(names, sizes) if s]
    assert kernels > 100
    assert not spilled, spilled
