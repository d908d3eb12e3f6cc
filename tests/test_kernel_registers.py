"""What the compiler says of the built kernels: the fused attention kernels of the default scheme keep their values in vector registers.
(A kernel that spills some stores them to memory and waits for them again, which no result shows.)"""
import struct

import pytest

pytest.importorskip("torch")
msgpack = pytest.importorskip("msgpack")

from paper_2504_02211_amd import ftattn

EM_AMDGPU, SHT_NOTE, NT_AMDGPU_METADATA = 224, 7, 32


def built_kernels(path):
    """Name -> metadata of every kernel in the code objects that the library carries."""
    with open(path, "rb") as f:
        blob = f.read()
    kernels, at = {}, blob.find(b"\x7fELF", 1)
    while at > 0:
        if struct.unpack_from("<H", blob, at + 18)[0] == EM_AMDGPU:
            sections, size, count = struct.unpack_from("<Q", blob, at + 40)[0], *struct.unpack_from("<HH", blob, at + 58)
            for header in range(at + sections, at + sections + size * count, size):
                if struct.unpack_from("<I", blob, header + 4)[0] != SHT_NOTE:
                    continue
                offset, length = struct.unpack_from("<QQ", blob, header + 24)
                note = at + offset
                while note < at + offset + length:
                    n_name, n_desc, kind = struct.unpack_from("<III", blob, note)
                    desc = note + 12 + (n_name + 3) // 4 * 4
                    if kind == NT_AMDGPU_METADATA:
                        for k in msgpack.unpackb(blob[desc:desc + n_desc], strict_map_key=False)["amdhsa.kernels"]:
                            kernels[k[".name"]] = k
                    note = desc + (n_desc + 3) // 4 * 4
        at = blob.find(b"\x7fELF", at + 1)
    return kernels


def test_attention_kernels_spill_no_vector_registers():
    kernels = built_kernels(ftattn.LIB_PATH)
    # ftattn_main<D, FT, CAUSAL, INJ, PS, SPLIT, SELF>: verification with duplication and with one class per row (PS 2 and 3) have more values than registers
    main = {n: k for n, k in kernels.items() if "ftattn_main" in n and "ELi2E" not in n and "ELi3E" not in n}
    assert len(main) >= 16 + 8 + 8 and sum("Lb0ELb1EEE" in n for n in main) == 8
    assert {n for n, k in main.items() if k[".vgpr_spill_count"]} == set()
