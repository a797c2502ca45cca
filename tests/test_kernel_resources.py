"""What the compiler gave the library's kernels, read from the metadata of the code object built from csrc/."""
import struct

import msgpack
import pytest

import paper_2506_01352_amd as tahq


def _kernels():
    """(name, metadata) of every kernel in the library's gfx950 code objects (ELF files inside the host library)."""
    blob = open(tahq.library_path(), "rb").read()
    found = []
    at = blob.find(b"\x7fELF", 4)
    while at >= 0:
        e_machine, = struct.unpack_from("<H", blob, at + 18)
        if blob[at + 4] == 2 and e_machine == 224:               # 64 bits, AMDGPU
            shoff, = struct.unpack_from("<Q", blob, at + 0x28)
            shentsize, shnum = struct.unpack_from("<HH", blob, at + 0x3A)
            for i in range(shnum):
                header = at + shoff + i * shentsize
                kind, = struct.unpack_from("<I", blob, header + 4)
                if kind != 7:                                    # notes
                    continue
                offset, size = struct.unpack_from("<QQ", blob, header + 0x18)
                pos, end = at + offset, at + offset + size
                while pos + 12 <= end:
                    namesz, descsz, ntype = struct.unpack_from("<III", blob, pos)
                    desc = pos + 12 + (namesz + 3) // 4 * 4
                    if ntype == 32 and blob[pos + 12:pos + 18] == b"AMDGPU":
                        meta = msgpack.unpackb(blob[desc:desc + descsz], raw=False, strict_map_key=False)
                        found.extend((k[".name"], k) for k in meta["amdhsa.kernels"])
                    pos = desc + (descsz + 3) // 4 * 4
        at = blob.find(b"\x7fELF", at + 4)
    return found


@pytest.fixture(scope="module")
def kernels():
    k = dict(_kernels())
    assert len(k) > 300, "no code object found in the library"
    return k


def test_no_kernel_needs_scratch_memory(kernels):
    assert not [n for n, k in kernels.items() if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]]


def test_allocation_tile_entropies_keep_their_wavefronts(kernels):
    # wavefronts per vector unit: 512 registers, in steps of eight
    for G, wavefronts in ((8, 8), (16, 8), (32, 7), (64, 4), (128, 2)):
        name, = [n for n in kernels if f"k_alloc_entropyILi{G}ELb1E" in n]
        assert 512 // (-(-kernels[name][".vgpr_count"] // 8) * 8) >= wavefronts, name


def test_every_kernel_is_in_the_library_once():
    # the library is linked of several code objects; a kernel that a shared header defines would be in each
    names = [name for name, _ in _kernels()]
    assert len(names) > 300 and len(set(names)) == len(names)
