"""Registers that the compiler could not hold: what a kernel spills it writes to memory and reads back, in every lane.  The built
library's own metadata says how much that is."""
import struct

import msgpack
import pytest

from paper_2511_00855_amd import binding as B


def _kernels():
    """The metadata of every kernel of the library: notes of the code objects in its offload bundles."""
    b = open(B.LIB_PATH, "rb").read()
    at = b.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        entries, p = struct.unpack_from("<Q", b, at + 24)[0], at + 32
        for _ in range(entries):
            off, size, name = struct.unpack_from("<QQQ", b, p)
            target, p = b[p + 24:p + 24 + name], p + 24 + name
            elf = b[at + off:at + off + size]
            if not target.startswith(b"hip") or elf[:4] != b"\x7fELF":
                continue
            phoff, (phsize, phnum) = struct.unpack_from("<Q", elf, 32)[0], struct.unpack_from("<HH", elf, 54)
            for h in range(phnum):
                kind, _, start, _, _, length = struct.unpack_from("<IIQQQQ", elf, phoff + h * phsize)
                n = start
                while kind == 4 and n < start + length:   # PT_NOTE
                    ns, ds, typ = struct.unpack_from("<III", elf, n)
                    desc = n + 12 + (ns + 3) // 4 * 4
                    if typ == 32:                         # NT_AMDGPU_METADATA
                        yield from msgpack.unpackb(elf[desc:desc + ds], strict_map_key=False).get("amdhsa.kernels", [])
                    n = desc + (ds + 3) // 4 * 4
        at = b.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)


@pytest.mark.parametrize("kernel", ["k_gram_lists", "k_refineI"])
def test_kernels_that_must_not_spill(kernel):
    found = [k for k in _kernels() if kernel in k[".name"]]
    assert found
    for k in found:   # a few registers that are written once outside the loops do not count
        assert k[".vgpr_spill_count"] <= 4 and k[".private_segment_fixed_size"] <= 16, (k[".name"], k[".vgpr_spill_count"], k[".private_segment_fixed_size"])


def test_static_arrays_of_the_search_are_what_its_launch_reckons_with():
    """How many workgroups a compute unit holds is reckoned from the dynamic LDS, the look-up tables (384 or 1,536 slots of 8 bytes) and
    at most 320 bytes of other static arrays."""
    found = [k for k in _kernels() if "k_searchI" in k[".name"]]
    assert found
    for k in found:
        tables = 1536 * 8 if k[".group_segment_fixed_size"] > 8192 else 384 * 8
        assert 0 <= k[".group_segment_fixed_size"] - tables <= 320, k[".name"]
