"""What the compiler made of the kernels, read from the metadata of the built library (no GPU): LDS of the general tiles
is their two operand buffers and nothing else, so that two blocks (four of the small ones) fit a CU, and no kernel keeps
a per-lane array in memory."""
import os
import re
import struct

import msgpack
import pytest


@pytest.fixture(scope="module")
def kernels():
    """{symbol: metadata} of every kernel in the code objects embedded in libxmoe.so."""
    from paper_2508_13337_amd import _lib
    if not os.path.exists(_lib.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    blob = open(_lib.LIB_PATH, "rb").read()
    out = {}
    for m in re.finditer(rb"\x7fELF\x02\x01", blob):
        elf = blob[m.start():]
        if struct.unpack_from("<H", elf, 18)[0] != 224:          # EM_AMDGPU
            continue
        phoff, = struct.unpack_from("<Q", elf, 32)
        phentsize, phnum = struct.unpack_from("<HH", elf, 54)
        for i in range(phnum):
            kind, _, at, _, _, size = struct.unpack_from("<IIQQQQ", elf, phoff + i * phentsize)
            if kind != 4:                                        # PT_NOTE
                continue
            end = at + size
            while at < end:
                n_name, n_desc, note = struct.unpack_from("<III", elf, at)
                at += 12
                name = elf[at:at + n_name]
                at += (n_name + 3) & ~3
                if name == b"AMDGPU\0" and note == 32:           # NT_AMDGPU_METADATA
                    meta = msgpack.unpackb(elf[at:at + n_desc], raw=False)
                    out.update({k[".name"]: k for k in meta["amdhsa.kernels"]})
                at += (n_desc + 3) & ~3
    assert len(out) > 50
    return out


def test_general_tiles_use_their_operand_buffers_only(kernels):
    tiles = {n: k for n, k in kernels.items() if "_mfma_kernel" in n and "gate_bwd" not in n}
    assert len(tiles) >= 30
    for n, k in tiles.items():
        # 128 threads: two buffers of (64 + 64) x 128 bytes; 256 threads: of (128 + 128) x 128
        want = 32768 if k[".max_flat_workgroup_size"] == 128 else 65536
        assert k[".group_segment_fixed_size"] == want, (n, k[".group_segment_fixed_size"])


def test_no_spills_outside_the_dact_epilogue(kernels):
    # (the 256-row dAct kernel holds its whole epilogue in registers and spills a few)
    spilled = {n: k[".private_segment_fixed_size"] for n, k in kernels.items()
               if k[".private_segment_fixed_size"] and "ffn_rowgemm_dma_kernel" not in n}
    assert not spilled, spilled
