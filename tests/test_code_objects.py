"""CPU check of the built library's kernel metadata: no kernel spills registers to scratch memory except those listed.
Inside a K loop a spill is a trip through memory per iteration, and results do not show it."""
import os
import re
import struct

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
# a few bytes outside the main loop
SPILLS_ALLOWED = {"k_nested_conv_smallcin", "k_nested_gemm_skinny", "k_nested_gemm_skinny_batch"}
# the large kernel's form for channel counts that are no power of two (last template argument 2): five dwords at most
GENERAL_FORM = re.compile(r"k_nested_gemm_big\w+ELi2EEEv")


def kernels(path):
    """(name, scratch bytes per lane) of every kernel in the library's gfx950 code objects."""
    msgpack = pytest.importorskip("msgpack")
    with open(path, "rb") as f:
        data = f.read()
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := data.find(magic, at)) >= 0:
        count, = struct.unpack_from("<Q", data, at + len(magic))
        q = at + len(magic) + 8
        for _ in range(count):
            off, size, tlen = struct.unpack_from("<QQQ", data, q)
            triple, q = data[q + 24:q + 24 + tlen], q + 24 + tlen
            if not size or b"gfx950" not in triple:
                continue
            elf = data[at + off:at + off + size]
            phoff, = struct.unpack_from("<Q", elf, 32)
            phnum, = struct.unpack_from("<H", elf, 56)
            for i in range(phnum):
                kind, = struct.unpack_from("<I", elf, phoff + 56 * i)
                if kind != 4:                                  # PT_NOTE
                    continue
                note, = struct.unpack_from("<Q", elf, phoff + 56 * i + 8)
                nlen, dlen, _ = struct.unpack_from("<III", elf, note)
                desc = note + 12 + (nlen + 3) // 4 * 4
                for k in msgpack.unpackb(elf[desc:desc + dlen])["amdhsa.kernels"]:
                    yield k[".name"], k[".private_segment_fixed_size"]
        at += len(magic)


def test_no_kernel_spills():
    lib = os.path.join(ROOT, "paper_2506_17870_amd", "libnq.so")
    if not os.path.exists(lib):
        from paper_2506_17870_amd import build
        build.build()
    seen, spilled = set(), []
    for name, scratch in kernels(lib):
        m = re.match(r"_ZN\d*\w*?(k_[a-z0-9_]+)", name)
        family = m.group(1) if m else name
        seen.add(family)
        if scratch and family not in SPILLS_ALLOWED and not (GENERAL_FORM.search(name) and scratch <= 20):
            spilled.append((name, scratch))
    assert {"k_nested_gemm_big", "k_nested_gemm", "k_nested_gemm_stat", "k_nested_gemm_slab"} <= seen
    assert not spilled, spilled
