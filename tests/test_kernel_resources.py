"""Registers of the built kernels, from the library's own metadata: the kernels
whose loops were measured without spills must stay so."""
import os
import re
import struct

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1702_00496_amd", "libatfd.so")
NT_AMDGPU_METADATA = 32


@pytest.fixture(scope="module")
def kernels():
    """name -> (registers, spilled registers, scratch bytes a lane) of every gfx950 kernel."""
    msgpack = pytest.importorskip("msgpack")
    data = open(LIB, "rb").read()
    out = {}
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        count, = struct.unpack_from("<Q", data, m.start() + 24)
        at = m.start() + 32
        for _ in range(count):
            off, size, length = struct.unpack_from("<QQQ", data, at)
            target = data[at + 24:at + 24 + length]
            at += 24 + length
            if b"gfx950" not in target or not size:
                continue
            elf = data[m.start() + off:m.start() + off + size]
            table, = struct.unpack_from("<Q", elf, 0x28)
            entry, number = struct.unpack_from("<HH", elf, 0x3a)
            for i in range(number):
                _, kind, _, _, start, _ = struct.unpack_from("<IIQQQQ", elf, table + i * entry)
                if kind != 7:   # a note section
                    continue
                namesz, descsz, note = struct.unpack_from("<III", elf, start)
                body = start + 12 + (namesz + 3) // 4 * 4
                if note == NT_AMDGPU_METADATA:
                    for k in msgpack.unpackb(elf[body:body + descsz], strict_map_key=False)["amdhsa.kernels"]:
                        out[k[".name"]] = (k[".vgpr_count"], k[".vgpr_spill_count"], k[".private_segment_fixed_size"])
    assert len(out) > 100
    return out


def test_streamed_ensemble_members_do_not_spill(kernels):
    found = {n: v for n, v in kernels.items() if "ens_stream_kernel" in n}
    assert len(found) == 4
    for name, (_, spilled, scratch) in found.items():
        assert spilled == 0 and scratch == 0, (name, spilled, scratch)
