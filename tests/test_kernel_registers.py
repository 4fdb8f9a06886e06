"""What the compiler gave the ring kernels, read from the metadata of the built library: kernels that are only worth having
where they stay in registers do."""
import struct

import msgpack
import pytest

from paper_2105_01827_amd.build import LIB

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _kernels():
    """(n, mangled name) -> metadata of every kernel that runs n / 8 threads a workgroup"""
    data, found, at = open(LIB, "rb").read(), {}, 0
    while (at := data.find(MAGIC, at)) >= 0:
        count, = struct.unpack_from("<Q", data, at + 24)
        entry = at + 32
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, entry)
            triple = data[entry + 24:entry + 24 + length]
            entry += 24 + length
            if b"gfx950" in triple:
                for k in _metadata(data[at + offset:at + offset + size])["amdhsa.kernels"]:
                    found[8 * k[".max_flat_workgroup_size"], k[".name"]] = k
        at += len(MAGIC)
    return found


def _metadata(elf):
    phoff, = struct.unpack_from("<Q", elf, 32)
    phsize, phnum = struct.unpack_from("<HH", elf, 54)
    for i in range(phnum):
        kind, _, offset, _, _, size = struct.unpack_from("<IIQQQQ", elf, phoff + i * phsize)
        if kind == 4:                      # PT_NOTE
            namesz, descsz, note = struct.unpack_from("<III", elf, offset)
            assert note == 32              # NT_AMDGPU_METADATA
            start = offset + 12 + (namesz + 3 & ~3)
            return msgpack.unpackb(elf[start:start + descsz])
    raise AssertionError("no metadata")


@pytest.fixture(scope="module")
def kernels():
    found = _kernels()
    assert {n for n, name in found if "perm_accumulate_ring" in name} == {1024, 2048, 4096, 8192}
    return found


def test_hoisted_decomposition_spills_nothing(kernels):
    for (n, name), k in kernels.items():
        if "decperm" in name and "ring" in name:
            assert k[".private_segment_fixed_size"] == 0, (n, name)


@pytest.mark.parametrize("weights,blocks,scratch", [(1, 0, 224), (0, 1, 280), (0, 0, 240)])
def test_perm_spills_at_n8192(kernels, weights, blocks, scratch):
    """There 128 registers do not hold everything; the bounds are bytes a lane."""
    found = [k for (n, name), k in kernels.items()
             if n == 8192 and f"perm_accumulate_ringILb1ELb{weights}ELb{blocks}E" in name]
    assert len(found) == 1 and found[0][".private_segment_fixed_size"] <= scratch


def test_masks_at_n8192_do_not_hold_a_whole_transform(kernels):
    """The constants of the small plaintext transform held all at once took 72 bytes a lane of a layer without rotations."""
    found = [k for (n, name), k in kernels.items() if n == 8192 and "scmult_masked_ring" in name]
    assert len(found) == 1 and found[0][".private_segment_fixed_size"] <= 64


@pytest.mark.parametrize("n", [1024, 2048, 4096, 8192])
def test_large_layers_without_rotations_leave_room_for_four_wavefronts(kernels, n):
    """One form of each ring, and of both widths below n = 4096, has at most 128 registers and spills none of them (to
    60 bytes a lane at n = 8192)."""
    fits = {"ILb1E" in name for (m, name), k in kernels.items() if m == n and "scmult_masked_ring" in name and
            k[".vgpr_count"] <= 128 and k[".private_segment_fixed_size"] <= (60 if n == 8192 else 0)}
    assert fits == ({True, False} if n < 4096 else {True})


@pytest.mark.parametrize("weights,blocks", [(1, 0), (0, 1), (0, 0)])
@pytest.mark.parametrize("kernel,few", [("perm_accumulate_ring", "Lb0E"), ("perm_accumulate_special_ring", "")])
def test_masks_behind_rotations_leave_their_scalars_alone(kernels, kernel, few, weights, blocks):
    """What a mask needs of the arguments is read behind the rotations.  Kept through them it took 46 to 64 more
    scalar registers than there are, in lanes of vector registers."""
    form = f"{kernel}ILb1ELb{weights}ELb{blocks}E{few}"
    plain, behind = ([k for (n, name), k in kernels.items() if n == 4096 and f"{form}Lb{mask}E" in name] for mask in (0, 1))
    assert len(plain) == len(behind) == 1
    assert behind[0][".sgpr_spill_count"] <= plain[0][".sgpr_spill_count"] + 12
    # they are read as a struct of the arguments: in order, structs at multiples of 16 bytes
    end = 0
    for arg in behind[0][".args"]:
        if arg[".value_kind"] != "by_value":
            break
        align = 4 if arg[".size"] == 4 else 16
        assert arg[".offset"] == -(-end // align) * align
        end = arg[".offset"] + arg[".size"]


@pytest.mark.parametrize("weights,blocks", [(1, 0), (0, 1), (0, 0)])
def test_small_launches_of_rotations_spill_nothing(kernels, weights, blocks):
    found = {n: k for (n, name), k in kernels.items() if n < 8192 and f"perm_accumulate_ringILb1ELb{weights}ELb{blocks}ELb1ELb0E" in name}
    assert set(found) == {1024, 2048, 4096}
    assert all(k[".private_segment_fixed_size"] == 0 for k in found.values()), {n: k[".vgpr_spill_count"] for n, k in found.items()}
