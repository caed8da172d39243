"""A vector instruction that takes another one's carry or lane mask out of VCC has to come two wait states after it on gfx950: the compiler
keeps them in what it forms itself, not inside a block of inline assembly.  Looks at the machine code of the built library."""
import os
import re
import struct
import subprocess

import pytest

from paper_2605_06113_amd import binding

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
CARRY_OUT = re.compile(r"v_(add|sub|subrev|addc|subb|subbrev)_co")


def _code_objects(path):
    """The gfx950 code objects of an offload bundle per translation unit (header: magic, number of entries; entry: offset, size, length
    of its name, name)."""
    data, magic = open(path, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        (entries,), q = struct.unpack_from("<Q", data, at + 24), at + 32
        for _ in range(entries):
            offset, size, length = struct.unpack_from("<QQQ", data, q)
            if b"gfx950" in data[q + 24:q + 24 + length]:
                yield data[at + offset:at + offset + size]
            q += 24 + length
        at = data.find(magic, at + 24)


def _too_early(lines):
    """(readers of VCC seen, those less than two wait states behind the vector instruction that wrote it) of straight code."""
    seen, bad, since, kernel, writer = 0, [], 2, "", ""
    for line in lines:
        if line.endswith(">:\n"):
            kernel, since = line, 2
            continue
        words = line.split("//")[0].replace(",", " ").split()
        if not words or not line[0].isspace():
            continue
        op, args = words[0], words[1:]
        if op == "s_nop":
            since += int(args[0], 0) + 1
        elif not op.startswith("v_"):
            since += 1
        else:
            if "vcc" in args[2:]:
                seen += 1
                if since < 2:
                    bad.append(f"{kernel.strip()} {writer} ; {' '.join(words)}")
            writes = (op.startswith("v_cmp") and args[0] == "vcc") or (CARRY_OUT.match(op) and args[1:2] == ["vcc"])
            since = 0 if writes else since + 1
            writer = " ".join(words) if writes else writer
    return seen, bad


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_no_vector_carry_is_read_too_early(tmp_path):
    binding.load()
    readers = 0
    for k, code in enumerate(_code_objects(binding.LIB_PATH)):
        path = tmp_path / f"{k}.co"
        path.write_bytes(code)
        run = subprocess.Popen([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", str(path)], stdout=subprocess.PIPE, text=True)
        seen, bad = _too_early(run.stdout)
        assert run.wait() == 0
        assert not bad, f"{len(bad)} of {seen}: {bad[:3]}"
        readers += seen
    assert readers > 1000  # (the pattern of such instructions fits this disassembler's text)
