"""Checks the machine code of kernels that load registers from inline assembly.

csrc/spmm_mfma.hpp issues its loads of B from inline assembly and waits for them with counts of its own,
while code that the compiler schedules runs.  The compiler takes the destinations for complete as soon as
the assembly has been issued; a copy of one, or a register given out again too early, would be a wrong
result now and then that no test shows reliably.  So the code itself is read: on every path, no instruction may
name a register that a load may still be about to write.
"""
from __future__ import annotations

import os
import re
import struct
import subprocess
import tempfile

_REGISTER = re.compile(r"\b([va])(?:(\d+)\b|\[(\d+):(\d+)\])")
_MEMORY = ("global_", "buffer_", "flat_", "scratch_")       # what vmcnt counts, stores too


def _registers(operands):
    found = set()
    for bank, one, first, last in _REGISTER.findall(operands):
        found.update((bank, i) for i in range(int(one or first), int(one or last) + 1))
    return found


class _Instruction:
    def __init__(self, line):
        text, _, note = line.partition("//")
        self.address = int(note.split(":")[0], 16)
        self.op, _, operands = text.strip().partition(" ")
        self.text = f"{self.op} {operands.strip()}"
        self.memory = self.op.startswith(_MEMORY)
        first, _, rest = operands.partition(",")
        load = self.memory and "_load_" in self.op
        self.loaded = _registers(first) if load else set()
        self.named = _registers(rest if load else operands)
        wait = re.search(r"vmcnt\((\d+)\)", operands) if self.op == "s_waitcnt" else None
        self.wait = int(wait.group(1)) if wait else None
        target = re.search(r"<[^>+]*(?:\+0x([0-9a-f]+))?>", note)
        self.target = int(target.group(1) or "0", 16) if target and "branch" in self.op else None


def hazards(lines, base=0):
    """Instructions of one disassembled kernel that name a register while a load into it may be in
    flight.  Kept for every register: how many memory instructions at least were issued after its load, over
    all paths (they complete in order, so vmcnt(N) ends the loads with N or more behind them)."""
    code = [_Instruction(line) for line in lines if "//" in line]
    at = {ins.address: i for i, ins in enumerate(code)}
    before = {0: {}}
    found, work = set(), [0]
    while work:
        i = work.pop()
        ins, flying = code[i], dict(before[i])
        if ins.op.startswith(("s_setpc", "s_swappc", "s_call")):
            raise RuntimeError(f"{ins.text}: calls are not followed")
        if ins.wait is not None:
            flying = {r: n for r, n in flying.items() if n < ins.wait}
        if ins.named & flying.keys():
            found.add(i)
        if ins.memory:
            flying = {r: min(n + 1, 64) for r, n in flying.items()}
            flying.update((r, 0) for r in ins.loaded)
        following = [] if ins.op in ("s_endpgm", "s_branch") else [i + 1]
        if ins.target is not None:
            following.append(at[base + ins.target])
        for j in following:
            if j >= len(code):
                continue
            known = before.get(j)
            if known is None:
                before[j] = dict(flying)
                work.append(j)
                continue
            earlier = {r: n for r, n in flying.items() if known.get(r, 65) > n}
            if earlier:
                known.update(earlier)
                work.append(j)
    return [code[i].text for i in sorted(found)]


def disassembly(library, rocm="/opt/rocm"):
    """{kernel: (address, lines)} of the gfx950 code in a HIP library."""
    tools = os.path.join(rocm, "llvm", "bin")
    with tempfile.TemporaryDirectory() as tmp:
        bundle, obj = os.path.join(tmp, "bundle"), os.path.join(tmp, "obj")
        subprocess.run([os.path.join(tools, "llvm-objcopy"), "--dump-section", ".hip_fatbin=" + bundle, library, os.devnull],
                       check=True)
        data = open(bundle, "rb").read()
        if not data.startswith(b"__CLANG_OFFLOAD_BUNDLE__"):
            raise RuntimeError(f"{library}: no code object bundle")
        pos = 32
        for _ in range(struct.unpack_from("<Q", data, 24)[0]):
            start, size, length = struct.unpack_from("<QQQ", data, pos)
            if b"gfx950" in data[pos + 24:pos + 24 + length]:
                open(obj, "wb").write(data[start:start + size])
            pos += 24 + length
        text = subprocess.run([os.path.join(tools, "llvm-objdump"), "-d", "--mcpu=gfx950", obj], check=True,
                              stdout=subprocess.PIPE, text=True).stdout
    kernels, lines = {}, []
    for line in text.splitlines():
        head = re.match(r"([0-9a-f]+) <(.*)>:$", line)
        if head:
            lines = []
            kernels[head.group(2)] = (int(head.group(1), 16), lines)
        else:
            lines.append(line)
    return kernels


def check(library, rocm="/opt/rocm"):
    """Raises if a matrix-core SpMM kernel of the library names a register with a load in flight; returns
    how many kernels were read."""
    kernels = {name: code for name, code in disassembly(library, rocm).items() if "spmm_mfma_kernel" in name}
    if not kernels:
        raise RuntimeError(f"{library}: no matrix-core SpMM kernel found")
    for name, (base, lines) in kernels.items():
        bad = hazards(lines, base)
        if bad:
            raise RuntimeError(f"{name}: {len(bad)} instructions name a register with a load in flight: " + "; ".join(bad[:4]))
    return len(kernels)
