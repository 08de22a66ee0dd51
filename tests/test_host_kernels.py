"""What the built kernels ask of a compute unit, from the metadata in the library: registers, LDS and arguments that a change in one
kernel's path would otherwise take from others unnoticed.  Needs no GPU."""
import struct

import msgpack
import pytest

import paper_2309_01507_amd as lpmm


def _kernels():
    """Metadata of every kernel in the library, by symbol."""
    with open(lpmm.lib_path(), "rb") as f:
        blob = f.read()
    out, at = {}, blob.find(b"AMDGPU\0\0")
    while at >= 0:                                       # ELF notes: name size, descriptor size, type; name; descriptor
        name_size, size, kind = struct.unpack_from("<3I", blob, at - 12)
        if name_size == 7 and kind == 32:
            for k in msgpack.unpackb(blob[at + 8:at + 8 + size], strict_map_key=False)["amdhsa.kernels"]:
                out[k[".name"]] = k
        at = blob.find(b"AMDGPU\0\0", at + 1)
    assert out, "no code object's metadata found"
    return out


@pytest.fixture(scope="module")
def kernels():
    return _kernels()


def _named(kernels, part):
    found = {n: k for n, k in kernels.items() if part in n}
    assert found, part
    return found


def test_the_quantizer_study_is_handed_what_it_uses(kernels):
    """A call on a small tensor takes little but its launch, and 260 more bytes of arguments were a fifth of it: the decompress kernel
    gets 16 entries, a compress kernel what its own rounding searches by."""
    explicit = lambda k: max(a[".offset"] + a[".size"] for a in k[".args"] if not a[".value_kind"].startswith("hidden"))
    for name, k in _named(kernels, "abl_dequant_kernel").items():
        assert k[".group_segment_fixed_size"] <= 64 and explicit(k) <= 160, name
    for part in ("abl_quant_block_kernel", "abl_quant_rank1_kernel"):
        for name, k in _named(kernels, part).items():
            # 88 bytes of addresses and sizes, three tables of 16 words, some scalars; the other rounding's tables would be 128 more
            assert explicit(k) <= 88 + 3 * 64 + 32, name


@pytest.mark.parametrize("part,waves", [("12phase_kernelILb0ELi1ELb1E", 6), ("12phase_kernelILb1ELi1ELb1E", 6),
                                        ("19factor_phase_kernelILb0ELi1ELb1E", 7), ("19factor_phase_kernelILb1ELi1ELb1E", 7)])
def test_first_passes_of_plain_plans_keep_their_waves(kernels, part, waves):
    """Plans by phases with rows of whole blocks only do not pay for the ragged statistics tiles' registers: six waves on a SIMD
    (rank-1) and seven (factorized) of 512 registers in steps of 8."""
    for name, k in _named(kernels, part).items():
        assert 512 // ((k[".vgpr_count"] + 7) // 8 * 8) >= waves and k[".private_segment_fixed_size"] == 0, (name, k[".vgpr_count"])
