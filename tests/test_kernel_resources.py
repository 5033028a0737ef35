"""Registers and scratch of the row movers that carry riders, read from the built library's own kernel metadata.

Every wave of a launch is given the registers and the scratch of the launch's hungriest path.  With 64 vector registers,
or with any scratch, the dispatcher refills the movers' wave slots more slowly: the stream of packet relays lost 3-17 % to
an index that had grown to that.  No GPU needed."""
import os
import struct
import subprocess

import msgpack
import pytest

from paper_2605_22428_amd import build

# kernels that move rows with an index or a plan riding along, and the scratch bytes a lane each may have.  (Instance 1
# of the dispatch's: the index for more than eight ids a token.  It spills a few registers; measured beside its movers
# it is ahead of a launch of its own.)
LEAN = {"k_relay_copy_index_next": 0, "k_relay_batch": 0, "k_relay_packets_copy_index_next": 0,
        "k_expand_index_nextILi0E": 0, "k_expand_index_nextILi1E": 24,
        "k_expand_index_plan_nextILi1ELb0ELi0E": 0, "k_expand_index_plan_nextILi1ELb0ELi1E": 24,
        "k_expand_index_plan_nextILi4ELb1ELi0E": 0, "k_expand_index_plan_nextILi4ELb0ELi1E": 24}


def _device_elf(path):
    """The gfx950 code object of a host library: clang's offload bundle in its .hip_fatbin section."""
    blob = open(path, "rb").read()
    at = blob.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        n, = struct.unpack_from("<Q", blob, at + 24)
        pos = at + 32
        for _ in range(n):
            off, size, name_len = struct.unpack_from("<QQQ", blob, pos)
            name = blob[pos + 24: pos + 24 + name_len].decode()
            pos += 24 + name_len
            if "gfx950" in name and size:
                yield blob[at + off: at + off + size]
        at = blob.find(b"__CLANG_OFFLOAD_BUNDLE__", pos)


def _kernels(elf):
    """The kernels' metadata: the msgpack map of the NT_AMDGPU_METADATA note (type 32)."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for i in range(shnum):
        _, kind, _, _, off, size = struct.unpack_from("<IIQQQQ", elf, shoff + i * shentsize)
        if kind != 7:
            continue
        pos = off
        while pos < off + size:
            name_size, desc_size, note = struct.unpack_from("<III", elf, pos)
            desc = pos + 12 + (name_size + 3) // 4 * 4
            if note == 32:
                yield from msgpack.unpackb(elf[desc: desc + desc_size], raw=False)["amdhsa.kernels"]
            pos = desc + (desc_size + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    path = build.LIB if os.path.exists(build.LIB) else build.build()
    return [k for elf in _device_elf(path) for k in _kernels(elf)]


@pytest.mark.parametrize("name", sorted(LEAN))
def test_row_movers_with_riders_stay_lean(kernels, name):
    found = [k for k in kernels if name in k[".name"]]
    assert found, "no kernel named %s in the library" % name
    for k in found:
        scratch, regs = k[".private_segment_fixed_size"], k[".vgpr_count"]
        assert scratch <= LEAN[name] and (LEAN[name] or regs < 64), (k[".name"], scratch, regs)
