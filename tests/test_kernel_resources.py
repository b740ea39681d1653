"""What the compiler gave the kernels, read from the metadata of the built library's code objects (no GPU)."""
import os
import struct

import pytest

import paper_2601_07396_amd as pkg

BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"
SHT_NOTE, NT_AMDGPU_METADATA = 7, 32


def _kernels(path):
    """Metadata of every kernel: each translation unit is a bundle of ELF files with one MessagePack note."""
    msgpack = pytest.importorskip("msgpack")
    with open(path, "rb") as f:
        d = f.read()
    out, at = {}, d.find(BUNDLE)
    while at >= 0:
        entry = at + 32
        for _ in range(struct.unpack_from("<Q", d, at + 24)[0]):
            offset, size, n = struct.unpack_from("<QQQ", d, entry)
            target, entry = d[entry + 24:entry + 24 + n], entry + 24 + n
            if b"amdgcn" not in target:
                continue
            elf = d[at + offset:at + offset + size]
            table, (width, count) = struct.unpack_from("<Q", elf, 0x28)[0], struct.unpack_from("<HH", elf, 0x3A)
            for i in range(count):
                _, kind, _, _, note, _ = struct.unpack_from("<IIQQQQ", elf, table + i * width)
                if kind != SHT_NOTE:
                    continue
                name, desc, tag = struct.unpack_from("<III", elf, note)
                if tag == NT_AMDGPU_METADATA:
                    start = note + 12 + (name + 3) // 4 * 4
                    for k in msgpack.unpackb(elf[start:start + desc])["amdhsa.kernels"]:
                        out[k[".name"]] = k
        at = d.find(BUNDLE, at + 1)
    return out


@pytest.mark.parametrize("kernel,least", [("project_stream_kernel", 100), ("forecast_mfma_kernel", 100)])
def test_streaming_kernels_use_no_scratch(kernel, least):
    """Kernels that stream rows through rings of registers: a ring that does not fit is written to memory and read back for every chunk
    of every row."""
    if not os.path.exists(pkg.lib_path()):
        pytest.skip("the library is not built")
    found = {n: k[".private_segment_fixed_size"] for n, k in _kernels(pkg.lib_path()).items() if kernel in n}
    assert len(found) >= least
    assert {n: bytes_ for n, bytes_ in found.items() if bytes_} == {}
