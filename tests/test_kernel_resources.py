"""Resources of the built kernels, from the metadata that the compiler writes
into this library's code objects (no GPU needed)."""
import os
import struct

import pytest

import paper_2507_02006_amd as pkg

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(data):
    """The gfx950 code objects of a library: one bundle per translation unit."""
    at = data.find(MAGIC)
    while at >= 0:
        n, p = struct.unpack_from("<Q", data, at + len(MAGIC))[0], at + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + idlen]
            p += 24 + idlen
            if b"gfx950" in name:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + 1)


def kernels(elf):
    """name -> metadata of the kernels of a code object (its AMDGPU note)."""
    msgpack = pytest.importorskip("msgpack")
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    shentsize, shnum = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(shnum):
        _, kind, _, _, off, size = struct.unpack_from("<IIQQQQ", elf, shoff + i * shentsize)
        if kind != 7:  # SHT_NOTE
            continue
        namesz, descsz, _ = struct.unpack_from("<III", elf, off)
        start = off + 12 + (namesz + 3) // 4 * 4
        meta = msgpack.unpackb(elf[start:start + descsz], raw=False, strict_map_key=False)
        return {k[".name"]: k for k in meta["amdhsa.kernels"]}
    return {}


def test_row_binning_uses_no_scratch_memory():
    """The bounds of the bins stay in the kernel arguments: a copy in scratch
    memory is read once per row and bin."""
    lib = os.path.join(os.path.dirname(pkg.__file__), "libaires.so")
    if not os.path.exists(lib):
        pytest.skip("library not built")
    with open(lib, "rb") as f:
        data = f.read()
    found = {}
    for elf in code_objects(data):
        found.update(kernels(elf))
    assert found, "no kernel metadata"
    bins = {n: k[".private_segment_fixed_size"] for n, k in found.items()
            if any(x in n for x in ("k_bin_count", "k_bin_scatter", "k_small_rows"))}
    assert len(bins) >= 5, bins
    assert not any(bins.values()), bins
