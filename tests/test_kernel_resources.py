"""Registers and shared memory of the kernels, from the metadata of the built library: what the dispatch rules and the comments at the
kernels count on."""
import os
import re
import struct

import msgpack
import pytest


@pytest.fixture(scope="module")
def kernels():
    from paper_2605_12396_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2605_12396_amd import build
        build.build()
    blob, found, at = open(binding.LIB_PATH, "rb").read(), {}, 0
    while (at := blob.find(b"AMDGPU\0\0", at + 1)) >= 0:         # ELF notes: name size, size, type, name, then a MessagePack map
        name_size, size, kind = struct.unpack_from("<III", blob, at - 12)
        if (name_size, kind) == (7, 32):
            for k in msgpack.unpackb(blob[at + 8:at + 8 + size])["amdhsa.kernels"]:
                m = re.match(r"_ZN2nz\d+(k_[a-z_]+?)(?:I((?:Li\d+E)+)E|E)", k[".name"])
                if m:
                    found[(m.group(1),) + tuple(int(x) for x in re.findall(r"Li(\d+)E", m.group(2) or ""))] = k
    return found


def test_adding_passes_keep_their_registers(kernels):
    """A workgroup of 512 threads has 128 registers a thread.  None of the passes spills any."""
    adding = {k: v for k, v in kernels.items() if k[0] == "k_decode" and k[1] in (2, 3, 4, 5, 6)}
    assert len(adding) >= 13
    for (_, mode, threads, delta), k in adding.items():
        assert k[".vgpr_spill_count"] == 0, (mode, threads, delta, k[".vgpr_spill_count"])


def workgroups_by_shared_memory(k):
    """Of a compute unit: 160 KB, given out in pieces of 1280 bytes."""
    return (160 << 10) // ((k[".group_segment_fixed_size"] + 1279) // 1280 * 1280)


def test_workgroups_of_a_compute_unit(kernels):
    """160 KB of shared memory and 512 registers a lane of a SIMD: three decompressing or staging workgroups of 256 threads, two of 512,
    two adding ones of 512."""
    for (_, mode, threads, delta), k in ((n, v) for n, v in kernels.items() if n[0] == "k_decode"):
        waves = threads // 64 // 4                                # of a workgroup, on each SIMD
        by_registers = 512 // ((k[".vgpr_count"] + 7) // 8 * 8) // waves
        resident = min(workgroups_by_shared_memory(k), by_registers)
        assert resident == (2 if threads == 512 else 3), (mode, threads, delta)


def test_encoder_workgroups_of_a_compute_unit(kernels):
    """Four of 256 threads, by registers: what a reduce's statistics blocks are cut for."""
    found = [k for n, k in kernels.items() if n[0] == "k_encode"]
    assert len(found) >= 11
    for k in found:
        by_registers = 512 // ((k[".vgpr_count"] + 7) // 8 * 8)
        assert min(workgroups_by_shared_memory(k), by_registers) == 4, k[".name"]


def test_large_alphabets_have_kernels_of_their_own(kernels):
    """k_decode's third parameter: bit 0 the predictor, bit 1 an alphabet whose codes take two bytes.  What its shorter rows save goes to its
    second-level tables, so that it fills the same shared memory."""
    shapes = {n[1:]: k[".group_segment_fixed_size"] for n, k in kernels.items() if n[0] == "k_decode"}
    small = [s for s in shapes if s[2] < 2]
    assert len(small) >= 21
    for mode, threads, form in small:
        assert abs(shapes[mode, threads, form + 2] - shapes[mode, threads, form]) <= 256, (mode, threads, form)
