"""What the bare barriers of the kernels rely on, read from the machine code of the built library (host only): the compiler does
not know of it, so a change of its order shows here."""
import os
import re
import struct
import subprocess

import pytest

from paper_2601_16238_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"
SOLO = "attn_bwd_dkdv_solo_kernel"


def code_objects():
    """The gfx950 code objects in the library."""
    data = open(build.LIB, "rb").read()
    at = data.find(BUNDLE)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + len(BUNDLE))
        entry = at + len(BUNDLE) + 8
        for _ in range(n):
            offset, size, name = struct.unpack_from("<QQQ", data, entry)
            if b"gfx950" in data[entry + 24:entry + 24 + name]:
                yield data[at + offset:at + offset + size]
            entry += 24 + name
        at = data.find(BUNDLE, at + 1)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{name: [(address, operation, operands, address that a branch goes to)]} of the kernels."""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(build.LIB):
        build.build()
    found = {}
    path = str(tmp_path_factory.mktemp("code") / "object")
    for obj in code_objects():
        names = {n.decode() for n in re.findall(rb"_ZN4attn\d+attn_\w+", obj)}
        names = [n for n in names if SOLO in n and not n.endswith("_kd")]
        if not names:
            continue
        with open(path, "wb") as f:
            f.write(obj)
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--disassemble-symbols=" + ",".join(names), path],
                              stdout=subprocess.PIPE, text=True, check=True).stdout
        for part in re.split(r"^[0-9a-f]+ <(?=\S+>:$)", text, flags=re.M)[1:]:
            name, body = part.split(">:\n", 1)
            found[name] = [parse(line) for line in body.splitlines() if "//" in line]
    assert found
    return found


def parse(line):
    code, note = line.split("//", 1)
    op, _, operands = code.strip().partition(" ")
    address = int(note.split(":")[0], 16)
    target = None
    if op.startswith(("s_cbranch", "s_branch")):
        words = int(operands) & 0xffff
        target = address + 4 + 4 * (words - 0x10000 if words & 0x8000 else words)
    return address, op, operands, target


def test_staging_space_is_read_before_the_ring_takes_it(kernels):
    """dK/dV by 64 keys a wave: K and V are sorted through ring positions that other waves' transfers fill behind the
    first barrier, which therefore has to find every LDS read of a wave done."""
    for name in (k for k in kernels if SOLO in k):
        reading, n_read = False, 0
        for _, op, operands, _ in kernels[name]:
            if op.startswith("ds_read"):
                reading, n_read = True, n_read + 1
            elif op == "s_waitcnt" and "lgkmcnt(0)" in operands:
                reading = False
            elif op == "s_barrier":
                break
        assert n_read >= 24 and not reading, name
