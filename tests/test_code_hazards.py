"""Wait states around the inline assembly of the kernels, read off the machine code of the built libraries (gfx950).

The hardware does not hold back an instruction for some of its operands: a number of other instructions or s_nop cycles (wait
states) has to lie between.  The compiler sees to that for the instructions it knows, but not inside inline assembly, so
whether such a block is safe can depend on what happened to be scheduled in front of it.  Each rule below is checked on every
path through every kernel: backwards from the instruction that reads to the one that wrote."""
import os
import re
import struct
import subprocess
import tempfile
from collections import defaultdict

import pytest

from paper_2405_05329_amd import build as kbuild

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(path):
    """The gfx950 code objects bundled in a host library."""
    with open(path, "rb") as f:
        data = f.read()
    at, found = data.find(BUNDLE), []
    while at >= 0:
        entries, p = struct.unpack_from("<Q", data, at + len(BUNDLE))[0], at + len(BUNDLE) + 8
        for _ in range(entries if entries < 8 else 0):   # (the bare text can also occur elsewhere)
            offset, size, length = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + length]:
                found.append(data[at + offset:at + offset + size])
            p += 24 + length
        at = data.find(BUNDLE, at + 1)
    return found


def registers(text):
    out = set()
    for m in re.finditer(r"(?<!\w)([sva])(?:\[(\d+):(\d+)\]|(\d+))(?!\w)", text):
        lo, hi = int(m[2] or m[4]), int(m[3] or m[4])
        out |= {m[1] + str(i) for i in range(lo, hi + 1)}
    return out | {r for r in ("vcc", "m0") if re.search(r"\b%s\b" % r, text)}


def scalar(regs):
    return {r for r in regs if r[0] == "s" or r == "vcc"}


class Instruction:
    def __init__(self, op, operands, at):
        self.op, self.at, self.text = op, at, f"{op} {operands}"
        ops = [o.strip() for o in re.split(r",(?![^\[]*\])", operands)] if operands else []
        self.valu = op.startswith("v_")
        self.vmem = op.startswith(("buffer_", "global_", "scratch_", "flat_"))
        self.to_lds = self.vmem and ("_lds_" in op or operands.endswith(" lds"))
        written = 1
        if self.valu and re.search(r"_co_u32|div_scale|_swap", op):
            written = 2
        elif self.to_lds or (self.vmem and re.search(r"store|atomic", op)) or \
                op.startswith(("ds_write", "s_cmp", "s_bitcmp", "s_cbranch", "s_branch", "s_waitcnt", "s_nop", "s_barrier")):
            written = 0
        self.defs = set().union(*map(registers, ops[:written]))
        self.uses = set().union(*map(registers, ops[written:]))
        self.wait_states = 1 + (int(ops[0], 0) if op == "s_nop" else 0)
        self.target = None
        if op.startswith(("s_cbranch", "s_branch")):
            offset = int(ops[0].split()[0], 0)
            self.target = at + 4 + 4 * (offset - 65536 if offset >= 32768 else offset)


def kernels(path):
    """{name: [Instruction, ...]} of every kernel in a library."""
    out = defaultdict(list)
    for obj in code_objects(path):
        with tempfile.NamedTemporaryFile(suffix=".co") as f:
            f.write(obj)
            f.flush()
            text = subprocess.run([OBJDUMP, "-d", f.name], capture_output=True, text=True, check=True).stdout
        name = None
        for line in text.splitlines():
            m = re.match(r"^[0-9a-f]+ <(\S+)>:", line)
            if m:
                name = m[1]
            m = re.match(r"^\s+(\S+)\s*(.*?)\s*// ([0-9A-F]{12}): ", line)
            if m and name:
                out[name].append(Instruction(m[1], m[2], int(m[3], 16)))
    return out


def violations(code, reads, writes, needed):
    """(states, writer, reader) for every path on which fewer than `needed` wait states lie between an instruction that
    `writes` holds for and a later one that reads, by `reads`, a register of it."""
    index, before = {i.at: n for n, i in enumerate(code)}, defaultdict(list)
    for n, i in enumerate(code):
        if i.target in index:
            before[index[i.target]].append(n)
        if n + 1 < len(code) and i.op not in ("s_branch", "s_endpgm", "s_setpc_b64"):
            before[n + 1].append(n)
    found = []
    for n, reader in enumerate(code):
        todo, seen = [(p, 0, frozenset(reads(reader))) for p in before[n]], set()
        while todo:
            p, states, regs = todo.pop()
            if not regs or states >= needed or (p, states, regs) in seen:
                continue
            seen.add((p, states, regs))
            writer = code[p]
            if writer.defs & regs and writes(writer):
                found.append((states, writer.text, reader.text))
                continue
            todo += [(q, states + writer.wait_states, regs - writer.defs) for q in before[p]]
    return found


RULES = {
    # a vector instruction writes a scalar register (v_readfirstlane, a spilled one coming back), a memory instruction reads it
    "vector-written scalar -> memory": (lambda i: scalar(i.uses) if i.vmem else (), lambda i: i.valu, 5),
    # a vector instruction writes a scalar register (a comparison's mask), another vector instruction reads it
    "vector-written scalar -> vector": (lambda i: scalar(i.uses) if i.valu else (), lambda i: i.valu, 2),
    # a matrix product's result, read by anything but another one (eight is what the compiler keeps behind the 16x16x32 form)
    "matrix product -> vector or memory": (lambda i: {r for r in i.uses if r[0] in "va" and r != "vcc"}
                                           if "mfma" not in i.op and (i.valu or i.vmem or i.op.startswith("ds_")) else (),
                                           lambda i: "mfma" in i.op, 8),
    # the LDS address of a load straight into LDS
    "m0 -> load to LDS": (lambda i: {"m0"} if i.to_lds else (), lambda i: not i.valu, 1),
}


@pytest.fixture(scope="module")
def libraries():
    libs = [p for p in (kbuild.LIB, kbuild.TRACE_LIB, kbuild.PROBE_LIB) if os.path.exists(p)]
    assert kbuild.LIB in libs
    return {os.path.basename(p): kernels(p) for p in libs}


@pytest.mark.parametrize("rule", RULES)
def test_wait_states(libraries, rule):
    checked = 0
    for lib, functions in libraries.items():
        for name, code in functions.items():
            found = violations(code, *RULES[rule])
            assert not found, f"{lib} {name}: {len(found)}, the first of them (states, writer, reader): {found[0]}"
            checked += any(RULES[rule][0](i) for i in code)
    assert checked >= 16, "every linear and attention kernel has such a reader"


def test_the_check_sees_what_it_is_for():
    code = [Instruction(op, operands, 4 * n) for n, (op, operands) in enumerate([
        ("v_readfirstlane_b32", "s6, v1"), ("s_cbranch_scc1", "2"), ("s_nop", "2"), ("s_nop", "0"),
        ("s_mov_b32", "m0, s9"), ("buffer_load_dwordx4", "v2, s[4:7], 0 offen lds")])]
    by_name = lambda rule: [v[0] for v in violations(code, *RULES[rule])]
    assert by_name("vector-written scalar -> memory") == [2]     # through the branch; 6 states along the other way
    assert by_name("m0 -> load to LDS") == [0]
