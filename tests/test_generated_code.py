"""What the hand-issued matrix instructions and the bare barriers of the kernels rely on, read from the machine code of the
built library (host only): the compiler does not know of either, so a change of its register allocation or order shows here."""
import os
import re
import struct
import subprocess

import pytest

from paper_2601_16238_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"
SOLO = "attn_bwd_dkdv_solo_kernel"
# v_mfma_f32_32x32x16 on gfx950: 8 passes of 4 cycles; the compiler keeps 12 wait states between one and the first other
# access to its result, and 2 between a vector instruction and a matrix instruction that takes its result as an operand
PASSES, RESULT, OPERAND = 8, 12, 2


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
    """{name: [(address, operation, operands, address that a branch goes to)]} of the kernels with hand-issued products."""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(build.LIB):
        build.build()
    found = {}
    path = str(tmp_path_factory.mktemp("code") / "object")
    for obj in code_objects():
        names = {n.decode() for n in re.findall(rb"_ZN4attn\d+attn_\w+", obj)}
        names = [n for n in names if not n.endswith("_kd") and
                 (SOLO in n or re.search("attn_(bwd_dkdv|bwd_pair|fwd_wide)_kernelILi256E", n)) and n + "\0" in obj.decode("latin1")]
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


def vector_registers(operands):
    out = set()
    for m in re.finditer(r"(?<![\w])v(?:\[(\d+):(\d+)\]|(\d+)\b)", operands):
        out.update(range(int(m[1]), int(m[2]) + 1) if m[1] else [int(m[3])])
    return out


class Wave:
    """Wait states that are still owed when an instruction issues; joins of paths keep the larger."""

    def __init__(self, result=(), operand=(), pipe=0):
        self.result, self.operand, self.pipe = dict(result), dict(operand), pipe

    def copy(self):
        return Wave(self.result, self.operand, self.pipe)

    def join(self, other):
        """Whether `other` owes more anywhere."""
        more = other.pipe > self.pipe
        self.pipe = max(self.pipe, other.pipe)
        for mine, theirs in ((self.result, other.result), (self.operand, other.operand)):
            for r, n in theirs.items():
                if n > mine.get(r, 0):
                    mine[r], more = n, True
        return more

    def passed(self, n):
        self.pipe = max(0, self.pipe - n)
        for owed in (self.result, self.operand):
            for r in [r for r, left in owed.items() if left <= n]:
                del owed[r]
            for r in owed:
                owed[r] -= n

    def issue(self, op, operands):
        """What is wrong with the instruction, or None."""
        wrong = None
        if op == "s_nop":
            self.passed(int(operands, 0) + 1)
            return None
        if op.startswith("v_mfma"):
            self.passed(self.pipe)
            to, a, b, c = [o.strip() for o in operands.split(", ")[:4]]
            touched = vector_registers(a + " " + b)
            if c != to:
                touched |= vector_registers(c) | vector_registers(to)
            # (one that accumulates onto the result of the one before needs no wait)
            if touched & set(self.result):
                wrong = "operands of a product are another's result"
            in_v = to.startswith("v")
            if in_v and (touched | vector_registers(c)) & set(self.operand):
                wrong = "operand from a vector instruction"
            self.passed(1)
            self.pipe = PASSES - 1
            if in_v:
                assert "32x32x16" in op
                self.result.update((r, RESULT) for r in vector_registers(to))
            return wrong
        if op.startswith(("v_", "ds_", "buffer_", "global_", "scratch_")):
            if vector_registers(operands) & set(self.result):
                wrong = "a product's result"
            self.passed(1)
            if op.startswith("v_"):
                self.operand.update((r, OPERAND) for r in vector_registers(operands.split(", ")[0]))
            return wrong
        self.passed(1)
        return None


def walk(code):
    """Every instruction along every path, until no path owes more than has been seen."""
    index = {ins[0]: i for i, ins in enumerate(code)}
    heads = {0} | {index[t] for *_, t in code if t is not None} | {i + 1 for i, ins in enumerate(code) if ins[3] is not None}
    seen, work, wrong = {0: Wave()}, [0], {}
    while work:
        i = work.pop()
        wave = seen[i].copy()
        while i < len(code):
            address, op, operands, target = code[i]
            problem = wave.issue(op, operands)
            if problem:
                wrong[address] = "%x: %s %s: %s" % (address, op, operands, problem)
            following = [] if op in ("s_branch", "s_endpgm") else [i + 1]
            if target is not None:
                following.append(index[target])
            if target is None and following and following[0] not in heads:
                i += 1
                continue
            for j in following:
                if j not in seen:
                    seen[j] = wave.copy()
                elif not seen[j].join(wave):
                    continue
                work.append(j)
            break
    return list(wrong.values())


def listing(*lines):
    return [(4 * i, *line.split(" ", 1), None) for i, line in enumerate(lines)]


def test_the_walk_finds_what_comes_too_early():
    product = "v_mfma_f32_32x32x16_bf16 v[0:15], v[16:19], v[20:23], v[0:15]"
    other = "v_mfma_f32_32x32x16_bf16 a[0:15], v[16:19], v[20:23], a[0:15]"
    read, operand = "v_exp_f32_e32 v40, v15", "v_mov_b32_e32 v16, v50"
    assert not walk(listing(product, "s_nop 11", read)) and walk(listing(product, "s_nop 10", read))
    assert not walk(listing(product, other, other, read)) and walk(listing(product, other, read))
    assert not walk(listing(product, product, "s_nop 15", "ds_write_b128 v60, v[12:15]"))
    assert walk(listing(product, "ds_write_b128 v60, v[12:15]")) and walk(listing(product, "v_mov_b32_e32 v3, 0"))
    assert not walk(listing(operand, "s_nop 1", product)) and walk(listing(operand, "s_nop 0", product))
    assert walk([(0, *product.split(" ", 1), None), (4, "s_cbranch_scc0", "2", 16), (8, "s_nop", "11", None),
                 (12, "s_nop", "0", None), (16, *read.split(" ", 1), None)])


def test_results_of_hand_issued_products_are_read_late_enough(kernels):
    assert sum(SOLO in k for k in kernels) == 16  # two widths, masks, with and without dS, element types
    for name, code in kernels.items():
        wrong = walk(code)
        assert not wrong, (name, wrong[:5])


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


def test_rows_leave_without_the_argument_block(kernels):
    """The launch of dK/dV and dQ side by side at D = 256 keeps more scalars than there are registers: none of the rows that it
    loads and stores may bring a spilled block of arguments back (16 lane reads a row, 1.2 us of a call of 13)."""
    found = {k: sum(op == "v_readlane_b32" for _, op, *_ in code) for k, code in kernels.items()
             if re.search("bwd_pair_kernelILi256ELi(192|256)ELb[01]ELb0E", k)}
    assert len(found) == 8 and max(found.values()) < 100, found
