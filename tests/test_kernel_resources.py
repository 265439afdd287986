"""What the compiled kernels hold of a CU, read from the metadata of the library built here: the launch shapes
and the two forms of the decoder rest on it, and no functional test would notice a change.
"""
import re
import struct
import subprocess

import msgpack
import pytest

from paper_2410_20650_amd import build

LDS_OF_A_CU = 160 * 1024
REGISTERS_OF_A_SIMD_LANE = 512


def code_object():
    with open(build.BUILT_LIB, "rb") as f:
        data = f.read()
    at = data.index(b"__CLANG_OFFLOAD_BUNDLE__")
    (entries,) = struct.unpack_from("<Q", data, at + 24)
    place = at + 32
    for _ in range(entries):
        offset, size, length = struct.unpack_from("<QQQ", data, place)
        if b"gfx950" in data[place + 24:place + 24 + length]:
            return data[at + offset:at + offset + size]
        place += 24 + length
    raise AssertionError("no gfx950 code object in the library")


def kernel_metadata(elf):
    """The AMDGPU metadata note (a msgpack map) of a 64-bit little-endian ELF file."""
    (sections_at,) = struct.unpack_from("<Q", elf, 0x28)
    entry_size, count = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(count):
        head = sections_at + i * entry_size
        (kind,) = struct.unpack_from("<I", elf, head + 4)
        offset, size = struct.unpack_from("<QQ", elf, head + 24)
        if kind != 7:       # SHT_NOTE
            continue
        name_size, desc_size, note = struct.unpack_from("<III", elf, offset)
        if note == 32:      # NT_AMDGPU_METADATA
            desc = offset + 12 + (name_size + 3) // 4 * 4
            return msgpack.unpackb(elf[desc:desc + desc_size], raw=False)["amdhsa.kernels"]
    raise AssertionError("no kernel metadata in the code object")


def symbol(elf, name):
    """Where a symbol's bytes are in the file, and how many."""
    sections_at, = struct.unpack_from("<Q", elf, 0x28)
    entry_size, count = struct.unpack_from("<HH", elf, 0x3A)
    sections = [struct.unpack_from("<IIQQQQIIQQ", elf, sections_at + i * entry_size) for i in range(count)]
    for _, kind, _, _, offset, size, link, _, _, entry in sections:
        if kind != 11:      # SHT_DYNSYM
            continue
        names = sections[link][4]
        for at in range(offset, offset + size, entry):
            text, _, _, home, value, length = struct.unpack_from("<IBBHQQ", elf, at)
            begin = names + text
            if elf[begin:elf.index(b"\0", begin)] == name.encode():
                return value - sections[home][3] + sections[home][4], length
    raise AssertionError(name)


def waves_of_a_simd(elf, name):
    """As many as the registers that the kernel's descriptor allocates leave room for (a limit that a kernel sets itself is kept by
    allocating more than it uses, which the metadata does not say)."""
    rsrc1, = struct.unpack_from("<I", elf, symbol(elf, name + ".kd")[0] + 48)
    return REGISTERS_OF_A_SIMD_LANE // (((rsrc1 & 63) + 1) * 8)


@pytest.fixture(scope="module")
def kernels():
    found = kernel_metadata(code_object())
    names = subprocess.run(["c++filt"], input="\n".join(k[".name"] for k in found), capture_output=True, text=True,
                           check=True).stdout.split("\n")
    short = [re.sub(r"\(.*", "", n).replace("void ", "").replace("nz::", "") for n in names]
    return {n: k for n, k in zip(short, found)}


def named(kernels, prefix):
    some = {n: k for n, k in kernels.items() if n.startswith(prefix)}
    assert some, prefix
    return some


def test_no_kernel_spills(kernels):
    for name, k in kernels.items():
        assert k[".private_segment_fixed_size"] == 0 and k[".vgpr_spill_count"] == 0, name


@pytest.mark.parametrize("prefix", ["decode_kernel<", "decode_direct_kernel<", "decode_batch_kernel<", "linear_batch_kernel<"])
def test_two_workgroups_of_eight_waves_share_a_cu(kernels, prefix):
    for name, k in named(kernels, prefix).items():
        assert k[".max_flat_workgroup_size"] == 512, name
        assert 2 * k[".group_segment_fixed_size"] <= LDS_OF_A_CU, name
        # two workgroups are four waves per SIMD
        assert k[".vgpr_count"] <= REGISTERS_OF_A_SIMD_LANE // 4, name


# One wave per tensor walks a ragged last chunk, and what that takes must not be held by all of them: binary32 and normalised tensors
# have as many waves as the walk of whole chunks allows.  The others, faster beyond the cache with fewer, have five, with gradients four.
@pytest.mark.parametrize("kind,least,most", [("true, -1, false, false, false", 6, 8), ("false, -1, true, false, false", 5, 8),
                                             ("false, 7, true, false, false", 5, 8), ("false, -1, false, false, false", 5, 5),
                                             ("false, -1, false, true, false", 5, 5), ("false, 7, false, false, false", 5, 5),
                                             ("false, 7, false, true, false", 5, 5), ("false, 3, false, false, false", 5, 5),
                                             ("false, 1, false, false, false", 5, 5), ("false, 0, false, false, false", 5, 5),
                                             ("false, 7, false, false, true", 4, 4)])
def test_waves_of_the_encoders(kernels, kind, least, most):
    k = kernels[f"encode_kernel<{kind}>"]
    assert least <= waves_of_a_simd(code_object(), k[".name"]) <= most, k[".vgpr_count"]
    # (workgroups of four waves: as many of them share a CU as a SIMD has waves)
    assert least * k[".group_segment_fixed_size"] <= LDS_OF_A_CU


def test_binary32_batches_of_many_workgroups_hold_one_group_of_turns(kernels):
    # (form 4, few workgroups, holds two groups: 8 fields and 16 lower halves more; form 0 walks whole states with one)
    of = {form: kernels[f"decode_batch_kernel<7, false, 1, {form}>"][".vgpr_count"] for form in (0, 2, 4)}
    assert of[2] <= of[0] + 8 and of[4] >= of[2] + 16, of


def test_weights_that_the_encoder_writes_back_leave_the_caches(kernels, tmp_path):
    # the call returns when the encoder has spoken, and says that the weights are there: stores at system scope in the walk of
    # whole chunks, a release at system scope behind that of the ragged one; no other encoder has either
    path = tmp_path / "code_object"
    path.write_bytes(code_object())
    of = {}
    for updates, kernel in enumerate(("encode_kernel<false, 7, false, false, false>", "encode_kernel<false, 7, false, false, true>")):
        name = kernels[kernel][".name"]
        of[updates] = subprocess.run(["/opt/rocm/llvm/bin/llvm-objdump", "-d", f"--disassemble-symbols={name}", str(path)],
                                     capture_output=True, text=True, check=True).stdout
        assert len(of[updates].split("\n")) > 1000, name
    through, release = r"buffer_store_dwordx4 .* sc0 sc1", r"buffer_wbl2 sc0 sc1"
    assert re.search(through, of[1]) and re.search(release, of[1])
    assert not re.search(through, of[0]) and not re.search(release, of[0])


def test_the_binary32_decoder_has_the_group_loop_of_a_ragged_chunk_once(kernels):
    # (with a copy for every source of the words it had 25752 bytes, and every launch took longer)
    assert symbol(code_object(), kernels["decode_kernel<7, false, 1, true>"][".name"])[1] <= 23500


def test_decoders_that_read_the_slot_table_carry_nothing_of_making_it(kernels):
    # last template argument: entry points or not (single tensors), the form of the walk (batches)
    table_and_words, steps = 16 * 1024 + 62 * 1024, 264 * 4
    for reading, making in (("decode_kernel<%s, false>", "decode_kernel<%s, true>"),
                            ("decode_batch_kernel<%s, 0>", "decode_batch_kernel<%s, 2>")):
        for kind in ("7, false, 0", "3, false, 0", "1, false, 0", "0, false, 0", "3, true, 0", "1, true, 0", "0, true, 0",
                     "7, false, 1", "7, false, 3"):
            lean, rich = kernels[reading % kind], kernels[making % kind]
            assert rich[".group_segment_fixed_size"] >= table_and_words + steps, kind
            # (k = 1 and 0 spread a field through a small table of their own, inside the words' window)
            assert lean[".group_segment_fixed_size"] <= table_and_words + 16, kind
            # the walk of a lossless or binary32 tensor needs about 80 registers, a lossy one about 50
            assert lean[".vgpr_count"] <= (88 if kind.startswith("7") else 58), (kind, lean[".vgpr_count"])
