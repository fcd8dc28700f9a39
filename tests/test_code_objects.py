"""The library's device code comes in objects small enough to load in passing (CPU only).

A process loads a code object when it first launches a kernel from it, in a time that grows with the object (one of
4.1 MB took a training process's first step from 3 to 13 ms), so the large families of kernels are split by what a
process uses (build.py, PARTS)."""
import struct

from paper_2509_20883_amd import recis as R

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
LIMIT = 1_500_000  # bytes


def device_code_objects(path):
    """(target, bytes) of every device entry of the library's offload bundles."""
    data = open(path, "rb").read()
    found, at = [], data.find(MAGIC)
    while at >= 0:
        (count,), pos = struct.unpack_from("<Q", data, at + len(MAGIC)), at + len(MAGIC) + 8
        for _ in range(count):
            _, size, name_len = struct.unpack_from("<QQQ", data, pos)
            found.append((data[pos + 24:pos + 24 + name_len].decode(), size))
            pos += 24 + name_len
        at = data.find(MAGIC, pos)
    return [(t, s) for t, s in found if not t.startswith("host")]


def test_code_objects_are_small():
    objs = device_code_objects(R.LIB_PATH)
    assert len(objs) >= 8 and all(t.endswith("gfx950") for t, _ in objs)
    assert max(s for _, s in objs) <= LIMIT, sorted((s for _, s in objs), reverse=True)
