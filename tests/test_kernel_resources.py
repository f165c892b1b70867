"""Registers and scratch of the built kernels, from the metadata the compiler leaves in the library (no GPU needed).

How many waves a SIMD holds is decided by a few registers: a launch with enough workgroups loses a third of its waves
where a change moves a kernel from 168 registers to 172, and no result shows it."""
import os
import re
import struct

import pytest

from paper_2506_11418_amd.build import LIB

msgpack = pytest.importorskip("msgpack")


def _metadata(elf: bytes):
    """The kernels of one code object: the msgpack note (type 32) of its ELF file."""
    shoff, shentsize, shnum = struct.unpack_from("<Q", elf, 40)[0], *struct.unpack_from("<HH", elf, 58)
    for i in range(shnum):
        kind, _, _, offset, size = struct.unpack_from("<IQQQQ", elf, shoff + i * shentsize + 4)
        at, end = offset, offset + size
        while kind == 7 and at < end:              # SHT_NOTE
            n_name, n_desc, note = struct.unpack_from("<III", elf, at)
            at += 12 + (n_name + 3) // 4 * 4
            if note == 32:
                yield from msgpack.unpackb(elf[at:at + n_desc])["amdhsa.kernels"]
            at += (n_desc + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(LIB):
        pytest.skip("the library is not built")
    data, found = open(LIB, "rb").read(), {}
    for at in (m.start() for m in re.finditer(b"\x7fELF", data)):
        if struct.unpack_from("<H", data, at + 18)[0] == 224:       # EM_AMDGPU
            for k in _metadata(data[at:]):
                found[k[".name"]] = (k[".vgpr_count"], k[".private_segment_fixed_size"])
    return found


def _instances(kernels, name):
    """Template arguments (types and numbers, as mangled) -> (registers, bytes of scratch a lane)."""
    got = {}
    for mangled, use in kernels.items():
        m = re.match(r"_ZN3ckv12_GLOBAL__N_1%d%sI(.*?)EEv" % (len(name), name), mangled)
        if m:
            got[tuple(re.findall(r"L[ib](\d+)E?|^(f|DF16b)", m.group(1) + "E"))] = use
    return {tuple(a or b for a, b in k): v for k, v in got.items()}


def test_bf16_attention_keeps_its_waves(kernels):
    found = _instances(kernels, "attn_mfma_kernel")
    assert len(found) == 2 * 4 * 2 * 2             # dims, heads per KV head, waves, strided and paged
    for (dim, heads, waves, paged), (registers, scratch) in found.items():
        three = paged == "0" or (dim, heads) == ("128", "8")
        assert scratch == 0 and registers <= (168 if three else 256), (dim, heads, waves, paged, registers, scratch)


def test_full_merges_hold_the_workgroups_per_cu_that_small_launches_are_cut_into(kernels):
    """Workgroups of four waves: one per CU for every wave a SIMD holds.  Registers come in eights, 512 a SIMD."""
    found = _instances(kernels, "merge_kernel")
    full = {k: v for k, v in found.items() if k[2] == "0"}
    assert len(full) == 2 * 2 * 2 * 2 + 4 * 2 * 2  # bf16: dims, capacities, pages, sinks; fp32: one kernel with and without sinks
    for (dtype, dim, _, capacity, paged, _), (registers, scratch) in full.items():
        waves = 512 // (-(-registers // 8) * 8)
        assert scratch == 0 and waves >= (4 if (dtype, paged) == ("f", "1") else 5), (dtype, dim, capacity, paged, registers, scratch)
    assert all(scratch == 0 for _, scratch in found.values())
