"""What the compiler's metadata in libfftconv.so says of the kernels; no device involved."""
import re
import struct

import msgpack

from paper_2311_05908_amd import fftconv


def code_objects(data):
    for at in (m.start() for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data)):
        entry = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            offset, size, length = struct.unpack_from("<QQQ", data, entry)
            if b"amdgcn" in data[entry + 24:entry + 24 + length]:
                yield data[at + offset:at + offset + size]
            entry += 24 + length


def kernels():
    """name -> metadata of every kernel of the library (the notes of its code objects)."""
    out = {}
    with open(fftconv.library_path(), "rb") as f:
        data = f.read()
    for elf in code_objects(data):
        table, size, count = struct.unpack_from("<Q", elf, 40)[0], *struct.unpack_from("<HH", elf, 58)
        for i in range(count):
            kind, offset = struct.unpack_from("<I", elf, table + i * size + 4)[0], struct.unpack_from("<Q", elf, table + i * size + 24)[0]
            if kind == 7 and elf[offset + 12:offset + 18] == b"AMDGPU":
                length = struct.unpack_from("<I", elf, offset + 4)[0]
                for k in msgpack.unpackb(elf[offset + 20:offset + 20 + length])["amdhsa.kernels"]:
                    out[k[".name"]] = k
    return out


def test_convolutions_of_the_row_kernels_use_no_scratch():
    rows = {n: k for n, k in kernels().items() if "k_row_conv" in n}
    assert len(rows) > 100
    assert {n: k[".private_segment_fixed_size"] for n, k in rows.items() if k[".private_segment_fixed_size"]} == {}


def test_kernels_that_form_rows_on_load_use_no_scratch():
    """Nor those of the same transforms from rows in memory: all are held to two workgroups of a compute unit by their registers."""
    names = "k_long_conv_rows", "k_long_rows_corr", "k_long_blocks_kf", "k_long_blocks_corr", "k_long_conv_blocks"
    long_rows = {n: k for n, k in kernels().items() if any(x in n for x in names)}
    assert all(any(x in n for n in long_rows) for x in names)
    assert {n: k[".private_segment_fixed_size"] for n, k in long_rows.items() if k[".private_segment_fixed_size"]} == {}
