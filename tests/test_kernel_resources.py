"""Registers of the built kernels whose residency the code relies on, from the metadata that the compiler leaves in the library.
No GPU."""
import re
import struct

import msgpack
import pytest

from paper_2402_10517_amd import binding as B

# the tile kernel over one tile and up to 8 batch rows: waves per SIMD by bit-width (512 registers, given out in eights)
WAVES = {3: 6, 4: 6, 5: 5, 6: 5, 7: 4, 8: 4}


def _kernels():
    """{mangled name: metadata} of every GPU kernel in the library (ELF objects for AMDGPU, machine 224, inside its file)."""
    data, out, pos = open(B.LIB_PATH, "rb").read(), {}, 0
    while (pos := data.find(b"\x7fELF", pos)) >= 0:
        if struct.unpack_from("<H", data, pos + 18)[0] == 224:
            sections, = struct.unpack_from("<Q", data, pos + 40)
            size, count = struct.unpack_from("<HH", data, pos + 58)
            for s in range(count):
                kind, = struct.unpack_from("<I", data, pos + sections + s * size + 4)
                note = pos + struct.unpack_from("<Q", data, pos + sections + s * size + 24)[0]
                if kind == 7:                                        # SHT_NOTE
                    name, desc, note_type = struct.unpack_from("<III", data, note)
                    if note_type == 32:                              # NT_AMDGPU_METADATA
                        start = note + 12 + (name + 3) // 4 * 4
                        for k in msgpack.unpackb(data[start:start + desc])["amdhsa.kernels"]:
                            out[k[".name"]] = k
        pos += 4
    return out


@pytest.mark.parametrize("kernel", ["list", "multi", "single"])
def test_one_tile_kernels_keep_their_waves_per_simd(kernel):
    pattern = {"list": r"gemv_tile_list_kernelILi(\d)E", "multi": r"gemv_tile_multi_kernelILi(\d)E",
               "single": r"gemv_tile_kernelILi(\d)ELi1ELi512ELb[01]ELb0E"}[kernel]
    seen = set()
    for name, k in _kernels().items():
        m = re.search(pattern, name)
        if m:
            b = int(m.group(1))
            seen.add(b)
            assert k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0, name
            assert 512 // ((k[".vgpr_count"] + 7) // 8 * 8) >= WAVES[b], "%s: %d registers" % (name, k[".vgpr_count"])
    assert seen == set(WAVES)


# the same kernel at batch 9 to 16 with one set of activation registers, with one and with two tiles per workgroup
WIDE_WAVES = {1: {3: 5, 4: 5, 5: 4, 6: 4, 7: 4, 8: 4}, 2: {3: 3, 4: 3, 5: 3, 6: 3, 7: 3, 8: 2}}


@pytest.mark.parametrize("tiles", [1, 2])
def test_kernels_for_nine_to_sixteen_batch_rows_keep_their_waves_per_simd(tiles):
    seen = set()
    for name, k in _kernels().items():
        m = re.search(r"gemv_tile_kernelILi(\d)ELi%dELi512ELb[01]ELb1ELb[01]ELb1E" % tiles, name)
        if m:
            b = int(m.group(1))
            seen.add(b)
            assert k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0, name
            assert 512 // ((k[".vgpr_count"] + 7) // 8 * 8) >= WIDE_WAVES[tiles][b], "%s: %d registers" % (name, k[".vgpr_count"])
    assert seen == set(WAVES)
