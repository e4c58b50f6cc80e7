"""Registers of the built kernels, from the code objects' own metadata: none may spill to
scratch memory.  The hot loops count the loads in flight to wait for single ones,
and a scratch reload among them waits for all."""
import os
import struct

import pytest

import paper_1711_07295_amd as ssj

msgpack = pytest.importorskip("msgpack")

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
LIB = os.path.join(os.path.dirname(ssj.__file__), "libssj.so")


def _code_objects(data):
    """The device code objects (ELF) of every offload bundle in `data`."""
    at = data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, p)
            target = data[p + 24:p + 24 + length]
            p += 24 + length
            if size and b"amdgcn" in target:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + 1)


def _kernels(elf):
    """The kernel descriptions in an ELF's AMDGPU metadata note."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    entsize, count = struct.unpack_from("<HH", elf, 58)
    for k in range(count):
        kind, = struct.unpack_from("<I", elf, shoff + k * entsize + 4)
        if kind != 7:  # SHT_NOTE
            continue
        at, size = struct.unpack_from("<QQ", elf, shoff + k * entsize + 24)
        end = at + size
        while at < end:
            n_name, n_desc, note = struct.unpack_from("<III", elf, at)
            name = at + 12
            desc = name + (n_name + 3) // 4 * 4
            if elf[name:name + 6] == b"AMDGPU" and note == 32:
                yield from msgpack.unpackb(elf[desc:desc + n_desc])["amdhsa.kernels"]
            at = desc + (n_desc + 3) // 4 * 4


def test_no_kernel_uses_scratch_memory():
    data = open(LIB, "rb").read()
    kernels = {k[".name"]: k for elf in _code_objects(data) for k in _kernels(elf)}
    assert sum("k_filter_mfma" in n for n in kernels) == 10
    assert {n: k[".private_segment_fixed_size"] for n, k in kernels.items()
            if k[".private_segment_fixed_size"]} == {}
