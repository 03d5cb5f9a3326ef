"""The denoise loop's kernels stay inside the 64 KB instruction cache that two compute units share, and keep everything in registers.
Code beyond the cache costs the loop some 25 us even where it is never run, and neither the compiler nor a parity test says so.
Read from the symbol tables of the library as built here."""
import struct

import pytest

from paper_2510_26742_amd import binding, build

INSTRUCTION_CACHE = 64 * 1024


def elf_sections(b):
    """(name, type, offset, size) of a 64-bit little-endian ELF file's sections."""
    shoff, = struct.unpack_from("<Q", b, 0x28)
    size, count, names = struct.unpack_from("<HHH", b, 0x3A)
    heads = [struct.unpack_from("<IIQQQQ", b, shoff + i * size) for i in range(count)]
    at = heads[names][4]
    return [(b[at + h[0]:b.index(b"\0", at + h[0])].decode(), h[1], h[4], h[5]) for h in heads]


def code_objects(library):
    """The gfx950 code objects in the library's offload bundles."""
    offset, size = next(s[2:] for s in elf_sections(library) if s[0] == ".hip_fatbin")
    fat = library[offset:offset + size]
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    start = fat.find(magic)
    while start >= 0:
        count, = struct.unpack_from("<Q", fat, start + len(magic))
        entry = start + len(magic) + 8
        for _ in range(count):
            at, n, length = struct.unpack_from("<QQQ", fat, entry)
            if b"gfx950" in fat[entry + 24:entry + 24 + length]:
                yield fat[start + at:start + at + n]
            entry += 24 + length
        start = fat.find(magic, entry)


def symbols(code):
    """name -> (value, size) of a code object's symbols."""
    sections = {s[0]: s[2:] for s in elf_sections(code)}
    at, size = sections[".symtab"]
    names = sections[".strtab"][0]
    out = {}
    for i in range(at, at + size, 24):
        name, _, _, _, value, n = struct.unpack_from("<IBBHQQ", code, i)
        out[code[names + name:code.index(b"\0", names + name)].decode()] = (value, n)
    return out


@pytest.fixture(scope="module")
def loop_kernels():
    binding.lib()   # says what to do if the library is missing
    with open(build.LIB, "rb") as f:
        library = f.read()
    return {k: v for code in code_objects(library) for k, v in symbols(code).items() if "expert_loop_kernel" in k}


# without a timeline (the form that pi0_denoise runs), with 8 and with 16 k steps per wave of the down projection
@pytest.mark.parametrize("down_steps", [8, 16])
def test_loop_kernel_fits_the_instruction_cache(loop_kernels, down_steps):
    stem = f"expert_loop_kernelILb0ELi{down_steps}EE"
    (name, (_, size)), = [(k, v) for k, v in loop_kernels.items() if stem in k and "." not in k]
    assert 0 < size <= INSTRUCTION_CACHE, (name, size)
    assert loop_kernels[name + ".private_seg_size"][0] == 0, "registers spilled"
    assert loop_kernels[name + ".num_vgpr"][0] <= 256
