"""What the compiler made of the kernels, read from the notes of the code objects inside the built library."""
import struct

import pytest

from paper_2409_15355_amd import binding as ba


def kernel_notes():
    """[(kernel, its metadata)] of every code object for the GPU in the library."""
    msgpack = pytest.importorskip("msgpack")
    ba.load()
    with open(ba.LIB_PATH, "rb") as f:
        lib = f.read()
    found, at = [], 0
    while (at := lib.find(b"\x7fELF", at + 1)) > 0:
        if struct.unpack_from("<H", lib, at + 18)[0] != 224:  # EM_AMDGPU
            continue
        shoff, = struct.unpack_from("<Q", lib, at + 40)
        shentsize, shnum = struct.unpack_from("<HH", lib, at + 58)
        for i in range(shnum):
            kind, _, _, offset, size = struct.unpack_from("<IQQQQ", lib, at + shoff + i * shentsize + 4)
            if kind != 7:  # SHT_NOTE
                continue
            name_size, desc_size, note = struct.unpack_from("<III", lib, at + offset)
            if note == 32 and desc_size <= size:  # NT_AMDGPU_METADATA
                desc = at + offset + 12 + (name_size + 3) // 4 * 4
                found += [(k[".name"], k) for k in msgpack.unpackb(lib[desc:desc + desc_size])["amdhsa.kernels"]]
    return found


def test_no_kernel_asks_for_scratch():
    kernels = kernel_notes()
    assert sum("attn_kernel" in name for name, _ in kernels) >= 10
    assert [(name, k[".private_segment_fixed_size"]) for name, k in kernels if k[".private_segment_fixed_size"]] == []


def test_small_encodes_fit_a_compute_unit_as_often_as_their_rule_reckons():
    """One launch per block row and KV head, a wave a SIMD each: four workgroups to a compute unit at head_dim 64, two at 128."""
    fresh = [(name, k) for name, k in kernel_notes() if "encode_short_kernel" in name and "EncodeFreshMeta" in name]
    assert len(fresh) == 4
    for name, k in fresh:
        most = 128 if "ILi64E" in name else 256
        assert k[".vgpr_count"] <= most and k[".max_flat_workgroup_size"] == 256, (name, k[".vgpr_count"])
