"""Registers of the built kernels (no GPU needed): kernels whose spills to
scratch memory were measured as lost time keep to what they were measured at."""
import os
import struct

import pytest

from paper_1903_04946_amd import soprop


def sections(elf):
    off, = struct.unpack_from("<Q", elf, 40)
    size, count, names = struct.unpack_from("<HHH", elf, 58)
    heads = [struct.unpack_from("<IIQQQQIIQQ", elf, off + i * size) for i in range(count)]
    base = heads[names][4]
    for h in heads:
        name = elf[base + h[0]:elf.index(b"\0", base + h[0])].decode()
        yield name, h[1], elf[h[4]:h[4] + h[5]]


@pytest.fixture(scope="module")
def kernels():
    """{mangled name: metadata} of every code object in the library."""
    msgpack = pytest.importorskip("msgpack")
    if not os.path.exists(soprop.LIB_PATH):
        import paper_1903_04946_amd.build as b
        b.build()
    out = {}
    with open(soprop.LIB_PATH, "rb") as f:
        library = f.read()
    bundle = next(data for name, _, data in sections(library) if name == ".hip_fatbin")
    at = bundle.find(b"\x7fELF")
    while at >= 0:
        for _, kind, data in sections(bundle[at:]):
            if kind != 7:  # SHT_NOTE
                continue
            owner, size, note = struct.unpack_from("<III", data)
            if note != 32:  # NT_AMDGPU_METADATA
                continue
            start = 12 + (owner + 3) // 4 * 4
            meta = msgpack.unpackb(data[start:start + size], strict_map_key=False)
            out.update((k[".name"], k) for k in meta["amdhsa.kernels"])
        at = bundle.find(b"\x7fELF", at + 4)
    assert out
    return out


def spills(kernels, *parts):
    found = {n: k[".vgpr_spill_count"] for n, k in kernels.items() if all(p in n for p in parts)}
    assert found, parts
    return found


def test_plane_pass_does_not_spill(kernels):
    assert not any(spills(kernels, "k3d_plane").values())


def test_two_fp64_surfaces_of_8192_points(kernels):
    """Plain runs and batch members (a kernel for runs with merged boundaries
    may spill more): 57 registers a lane when a substep took 14.6 us."""
    single = spills(kernels, "k1d_prop_kernelIdNS_5SchedILi8192E", "Li2ELi1E")
    assert min(single.values()) <= 57
    assert max(spills(kernels, "k1b_kernelIdNS_5SchedILi8192ELi8E", "Li2ELi1E").values()) <= 57


def test_batch_members_of_4096_points(kernels):
    """Two FP64 surfaces, exchanged together: 48 registers a lane when 32
    members took 401 us (105: 508)."""
    assert max(spills(kernels, "k1b_kernelIdNS_5SchedILi4096ELi8E", "Li2ELi2E").values()) <= 48


def test_trapezoid_of_8192_points(kernels):
    """One surface: 63 registers a lane when a solve took 26.9 ms (127: 33.6)."""
    assert max(spills(kernels, "k1d_trap_kernelINS_5SchedILi8192E", "Li1ELi1E").values()) <= 63
