"""Registers and LDS of the built kernels, from the metadata of the library's own code objects: what decides how many workgroups share a
CU.  CPU only."""
import struct

import msgpack
import pytest

from paper_2507_19131_amd import binding as M

LDS_UNIT, LDS_UNITS, SIMD_REGISTERS, REGISTER_GRANULE, MAX_WAVES = 1280, 128, 512, 8, 8


def _code_objects(data):
    at = data.find(b"\x7fELF", 4)
    while at >= 0:
        yield data[at:]
        at = data.find(b"\x7fELF", at + 4)


def _kernels(elf):
    """Metadata of the kernels of a code object: the note of type 32 named AMDGPU."""
    offset, = struct.unpack_from("<Q", elf, 0x28)
    entry, count = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, offset + i * entry + 4)
        start, size = struct.unpack_from("<QQ", elf, offset + i * entry + 0x18)
        at = start
        while kind == 7 and at < start + size:
            name, desc, note = struct.unpack_from("<III", elf, at)
            body = at + 12 + (name + 3) // 4 * 4
            if note == 32 and elf[at + 12:at + 12 + name].rstrip(b"\0") == b"AMDGPU":
                for k in msgpack.unpackb(elf[body:body + desc], raw=False)["amdhsa.kernels"]:
                    yield k[".name"], k
            at = body + (desc + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    M.load()
    with open(M.lib_path(), "rb") as f:
        data = f.read()
    found = {name: k for elf in _code_objects(data) for name, k in _kernels(elf)}
    assert len(found) > 100
    return found


def _window(NH, taps, scored, HG, QS, codes, magic, beside):
    b = lambda v: "Lb%dE" % v
    return "_ZN5mixaq13window_kernelILi%dE%s%sLi%dELi%dE%s%s%sEEvNS_4GeomENS_7WinArgsE" % (NH, b(taps), b(scored), HG, QS, b(codes), b(magic), b(beside))


def waves_per_simd(k):
    registers = -(-k[".vgpr_count"] // REGISTER_GRANULE) * REGISTER_GRANULE
    return min(MAX_WAVES, SIMD_REGISTERS // registers)


def lds_units(k):
    return -(-k[".group_segment_fixed_size"] // LDS_UNIT)


def workgroups_per_cu(k):
    waves = k[".max_flat_workgroup_size"] // 64
    return min(4 * waves_per_simd(k) // waves, LDS_UNITS // lds_units(k))


@pytest.mark.parametrize("scored", [0, 1])
@pytest.mark.parametrize("magic", [0, 1])
def test_forms_of_three_heads_beside_a_second_chain(kernels, scored, magic):
    """C = 96, two chains.  Pairs, up to 512 windows each: two workgroups a CU of the one, so that the other has none unless a third fits.
    One wave per head: five workgroups, which is what the launch has at its upper line."""
    assert workgroups_per_cu(kernels[_window(3, 0, scored, 1, 2, 0, magic, 1)]) == 3
    single = kernels[_window(3, 0, scored, 1, 1, 0, magic, 1)]
    assert workgroups_per_cu(single) == 5 and single[".vgpr_spill_count"] == 0


@pytest.mark.parametrize("magic", [0, 1])
@pytest.mark.parametrize("NH,HG,workgroups", [(4, 4, 4), (4, 6, 3), (8, 4, 2)])
def test_wide_forms_of_one_wave_per_head(kernels, NH, HG, workgroups, magic):
    """C = 512, 768 and 1024 beyond 256 workgroups of pairs: the workgroups a CU holds, by registers and by whole units of LDS, and no register in
    scratch memory."""
    k = kernels[_window(NH, 0, 0, HG, 1, 1, magic, 0)]
    assert workgroups_per_cu(k) == workgroups and k[".vgpr_spill_count"] == 0


def _token(NH, RB, steps):
    return "_ZN5mixaq12token_kernelILi%dELi%dELb0ELb%dEEEvNS_4GeomENS_7TokArgsE" % (NH, RB, steps)


@pytest.mark.parametrize("steps", [0, 1])
@pytest.mark.parametrize("NH,RB,workgroups", [(3, 1, 5), (4, 1, 4), (6, 1, 2), (8, 1, 2), (12, 1, 1), (12, 2, 1)])
def test_token_workgroups_of_a_cu(kernels, NH, RB, workgroups, steps):
    """As many with the table of steps as with the smaller one of cubics: what the registers hold."""
    k = kernels[_token(NH, RB, steps)]
    assert workgroups_per_cu(k) == 4 * waves_per_simd(k) // NH == workgroups


@pytest.mark.parametrize("scored,magic", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("steps", [0, 1])
def test_token_workgroups_beside_a_window_of_a_second_chain(kernels, steps, scored, magic):
    """C = 256: a CU's registers hold two token workgroups, or one beside a window workgroup of the other chain.  A token workgroup that lies behind
    a window workgroup leaves room for a second one behind itself; otherwise the CU has one until both are through."""
    window = kernels[_window(4, 0, scored, 2, 2, 0, magic, 0)]
    assert lds_units(window) + 2 * lds_units(kernels[_token(8, 1, steps)]) <= LDS_UNITS
