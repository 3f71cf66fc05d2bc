"""What the built kernels ask of the machine, from the metadata of the library's own code objects: a kernel that indexes an array
by a run-time value keeps it in scratch memory, which is a chain of stores and loads in every workgroup and raises no error."""
import struct

import pytest

import paper_2407_00611_amd as st

msgpack = pytest.importorskip("msgpack")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects():
    data = open(st.library_path(), "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        (n,), p = struct.unpack_from("<Q", data, at + len(MAGIC)), at + len(MAGIC) + 8
        for _ in range(n):
            offset, size, name = struct.unpack_from("<QQQ", data, p)
            p += 24 + name
            if b"gfx950" in data[p - name:p] and size:
                yield data[at + offset:at + offset + size]
        at = data.find(MAGIC, at + 1)


def _kernels():
    out = {}
    for elf in _code_objects():
        shoff, = struct.unpack_from("<Q", elf, 40)
        entry, count = struct.unpack_from("<HH", elf, 58)
        for i in range(count):
            _, kind, _, _, offset, size = struct.unpack_from("<IIQQQQ", elf, shoff + i * entry)
            if kind != 7:                                      # SHT_NOTE
                continue
            name, desc, _ = struct.unpack_from("<III", elf, offset)
            start = offset + 12 + (name + 3) // 4 * 4
            for k in msgpack.unpackb(elf[start:start + desc])["amdhsa.kernels"]:
                out[k[".name"]] = k
    return out


def test_no_kernel_keeps_its_arguments_in_scratch():
    kernels = _kernels()
    # beside the assembly, which owns all vector registers, one may have to wait in memory (8 bytes a lane, beside
    # the longer lists of the one walk two)
    for part, most in (("bwd_dkv_fast_kernel", 0), ("bwd_pair_fast_kernel", 8), ("bwd_dq_fast_kernel", 8), ("fwd_fast_kernel", 8),
                       ("bwd_one_kernel", 16), ("add_pairs_kernel", 0), ("add_kv_parts", 0), ("add_parts", 0), ("combine_kernel", 0)):
        found = {name: k for name, k in kernels.items() if part in name}
        assert found, part
        for name, k in found.items():
            assert k[".private_segment_fixed_size"] <= most, name
