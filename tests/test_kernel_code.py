"""The code of the product kernels as the compiler leaves it: where the assembler puts the entries of a table of patterns
(csrc/rsr_lib.hip, RSR_TABLE), and how large the kernels are."""
import os
import re
import struct
import subprocess

import pytest

from paper_2411_06360_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def functions(path):
    """The functions of the gfx950 code objects in a file that hipcc wrote: name -> code."""
    data, found = open(path, "rb").read(), {}
    for bundle in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        at, = struct.unpack_from("<Q", data, bundle.end())
        entry = bundle.end() + 8
        for _ in range(at):
            offset, size, name = struct.unpack_from("<QQQ", data, entry)
            target = data[entry + 24:entry + 24 + name]
            entry += 24 + name
            if b"gfx950" in target:
                found.update(functions_of(data[bundle.start() + offset:bundle.start() + offset + size]))
    return found


def functions_of(elf):
    start, = struct.unpack_from("<Q", elf, 0x28)
    size, count = struct.unpack_from("<HH", elf, 0x3A)
    sections = [struct.unpack_from("<IIQQQQIIQQ", elf, start + i * size) for i in range(count)]
    found = {}
    for section in sections:
        if section[1] != 2:  # SHT_SYMTAB
            continue
        names = sections[section[6]][4]
        for at in range(section[4], section[4] + section[5], 24):
            name, info, _, where, value, length = struct.unpack_from("<IBBHQQ", elf, at)
            if info & 15 == 2 and length:  # STT_FUNC
                code = sections[where][4] + value - sections[where][3]
                found[elf[names + name:elf.index(b"\0", names + name)].decode()] = elf[code:code + length]
    return found


def table_of(tmp_path, stride, store):
    """A kernel that holds one table of four positions whose "instructions" are words that say what they stand for."""
    source = open(os.path.join(ROOT, "paper_2411_06360_amd", "csrc", "rsr_lib.hip")).read()
    macro = re.search(r"#define RSR_TABLE\((?:.*\\\n)+.*\n", source).group(0)
    word = lambda x: f'" .long 0x{x:x}0000 + 256 * rsr_p + rsr_q\\n"'
    hip, obj = tmp_path / "table.hip", tmp_path / "table.o"
    hip.write_text("#include <hip/hip_runtime.h>\n" + macro + '__global__ void table() {\n  asm volatile(" s_endpgm\\n"\n'
                   f'    RSR_TABLE("t", 96, 4, {stride}, {word(0xA)}, {word(0xB)}, {word(0xC)}, {word(0xD) * store}, {word(0xE)}, "s[94:95]")::);\n}}\n')
    run = subprocess.run([build.hipcc(), "-O3", f"--offload-arch={build.ARCH}", "--cuda-device-only", "-c", "-o", str(obj), str(hip)],
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    return run, obj


@pytest.mark.parametrize("store", [1, 2, 3])
def test_patterns_lie_a_stride_apart_whatever_their_instructions_take(tmp_path, store):
    stride = 4 * (4 * (store + 1) + 5)
    run, obj = table_of(tmp_path, stride, store)
    assert run.returncode == 0, run.stdout
    (code,) = functions(obj).values()
    words = list(struct.unpack(f"<{len(code) // 4}I", code))
    first = words.index(0xA0000)  # pattern 0 begins with the gather of position 0
    for pattern in range(16):
        rows = [q for q in range(4) if not pattern >> q & 1]
        want = 0xA0000 + 256 * pattern + rows[0] if rows else 0xD0000 + 256 * pattern
        assert words[first + pattern * stride // 4] == want, pattern


def test_a_pattern_longer_than_the_stride_is_an_error(tmp_path):
    run, _ = table_of(tmp_path, 32, 2)
    assert run.returncode != 0 and ".org" in run.stdout, run.stdout


def test_every_kernel_is_within_reach_of_a_branch():
    """A short branch reaches 128 KB, and the compiler, which takes a .rept for a few instructions, plans no others."""
    if not os.path.exists(build.LIB):
        build.build()
    sizes = {name: len(code) for name, code in functions(build.LIB).items()}
    assert len(sizes) > 14 and max(sizes.values()) < 120 * 1024, sizes
