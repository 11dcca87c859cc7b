"""What the compiler made of kernels whose registers or code are at a limit, read from the built library: a change elsewhere in a source file
can tip them over, which costs time and no result shows it."""
import os
import struct

import pytest

ELF, BUNDLE = b"\x7fELF", b"__CLANG_OFFLOAD_BUNDLE__"


def sections(elf):
    """[(type, link, bytes)] of an ELF file's sections."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    size, count = struct.unpack_from("<HH", elf, 0x3A)
    got = []
    for i in range(count):
        _, kind, _, _, off, length, link = struct.unpack_from("<IIQQQQI", elf, shoff + i * size)
        got.append((kind, link, b"" if kind == 8 else elf[off:off + length]))
    return got


def code_objects(lib):
    at = lib.find(BUNDLE)
    while at >= 0:
        n, = struct.unpack_from("<Q", lib, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, name = struct.unpack_from("<QQQ", lib, p)
            if lib[p + 24:p + 24 + name].endswith(b"gfx950") and size:
                yield lib[at + off:at + off + size]
            p += 24 + name
        at = lib.find(BUNDLE, at + 1)


@pytest.fixture(scope="module")
def kernels():
    """Mangled name -> (bytes of code, bytes of scratch per lane, bytes of LDS beside what a launch asks for)."""
    from paper_2403_17312_amd import binding, build
    if not os.path.exists(binding.LIB_PATH):
        build.build()
    with open(binding.LIB_PATH, "rb") as f:
        lib = f.read()
    got = {}
    for elf in code_objects(lib):
        assert elf[:4] == ELF
        secs = sections(elf)
        headers = [struct.unpack_from("<IIQQQQ", elf, struct.unpack_from("<Q", elf, 0x28)[0] + i * struct.unpack_from("<H", elf, 0x3A)[0])
                   for i in range(len(secs))]
        for kind, link, data in secs:
            if kind != 2:                                 # the symbol table
                continue
            code, fixed = {}, {}
            for o in range(0, len(data), 24):
                name, info, _, sec, value, size = struct.unpack_from("<IBBHQQ", data, o)
                text = secs[link][2]
                sym = text[name:text.index(b"\0", name)].decode()
                if sym.endswith(".kd"):                   # kernel descriptor: LDS and scratch are its first words
                    _, _, _, addr, off, _ = headers[sec]
                    fixed[sym[:-3]] = struct.unpack_from("<II", elf, off + value - addr)
                elif info & 15 == 2:
                    code[sym] = size
            got.update({k: (code[k], fixed[k][1], fixed[k][0]) for k in fixed})
    return got


def seed_sums(dtype, d, tiles, rows):
    return f"_ZN3swa18swa_prefill_kernelINS_{len(dtype)}{dtype}ELi{d}ELi{tiles}ELb{int(rows)}ELi2EEEvNS_11PrefillArgsE"


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype", ["F16", "BF16"])
def test_column_sums_hold_a_tiles_work_twice_and_no_more(kernels, dtype, d):
    """16 bits: once with the mask and once without, where fp32 has two tiles in a round.  The kernel runs behind another one, so its code comes
    from memory; loops that the compiler copied for a value fixed in the launch made it up to twice as long."""
    for tiles in (1, 2, 3, 4):
        assert kernels[seed_sums(dtype, d, tiles, False)][0] <= 1.2 * kernels[seed_sums("F32", d, tiles, False)][0], tiles
    assert kernels[seed_sums(dtype, d, 1, True)][0] <= 1.2 * kernels[seed_sums("F32", d, 1, True)][0]


def test_fp32_column_sums_of_many_rows_spill_no_more(kernels):
    """97 to 128 rows at d = 128: 97 registers (376 bytes) do not fit; code that only 16 bits use made it 134 (412 bytes)."""
    assert kernels[seed_sums("F32", 128, 4, False)][1] <= 376
    for tiles in (1, 2, 3):
        assert kernels[seed_sums("F32", 128, tiles, False)][1] == 0, tiles


def test_1024_threads_leave_room_for_the_longest_caches(kernels):
    """The rule that gives long caches 1024 threads counts 14 KiB of the kernel's own LDS beside 20 bytes a slot of 7168."""
    seen = [k for k in kernels if k.startswith("_ZN3swa17swa_decode_kernelI") and "ELi1024ELb0E" in k]
    assert len(seen) == 6
    for k in seen:
        assert kernels[k][2] <= 14 * 1024, k
