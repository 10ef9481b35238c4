"""What the compiler does not check of the hand-written loads into LDS (csrc/gemm_tile.hpp: load_to_lds), looked up in the
gfx950 code of a built library.

Hazards inside inline assembly are the author's: a buffer load must not read a scalar register within five wait states
after a vector instruction wrote it (a lane read, a compare, a carry).  The kernels' descriptors are made by scalar
instructions, which the hardware waits for; whether they all still are depends on what the compiler does with the code
around, so every build looks.
"""

from __future__ import annotations

import os
import re
import struct
import subprocess
import tempfile

OBJDUMP = os.path.join(os.path.dirname(os.path.dirname(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"))), "llvm", "bin",
                       "llvm-objdump")
WAIT_STATES = 5
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(path: str):
    """The gfx950 code objects in a library or object file (the bundles that hipcc embeds, header by header)."""
    data = open(path, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + len(MAGIC))
        pos = at + len(MAGIC) + 8
        if n <= 64:   # the magic can also stand in a string
            for _ in range(n):
                offset, size, length = struct.unpack_from("<QQQ", data, pos)
                triple = data[pos + 24:pos + 24 + length]
                pos += 24 + length
                if b"gfx950" in triple and size:
                    yield data[at + offset:at + offset + size]
        at = data.find(MAGIC, at + len(MAGIC))


def listing(code: bytes) -> str:
    with tempfile.NamedTemporaryFile(suffix=".co") as f:
        f.write(code)
        f.flush()
        return subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", f.name], check=True, capture_output=True, text=True).stdout


def _registers(operand: str) -> set:
    m = re.fullmatch(r"s(\d+)", operand) or re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    if not m:
        return {106, 107} if operand == "vcc" else set()
    return set(range(int(m[1]), int(m[m.lastindex]) + 1))


def _vector_writes(op: str, args: list) -> set:
    """Scalar registers that a vector instruction writes."""
    if not op.startswith("v_") or not args:
        return set()
    if op.startswith(("v_readlane", "v_readfirstlane", "v_cmp")):
        return _registers(args[0])
    if re.search(r"_co_|_co_ci_|v_mad_[ui]64|v_div_scale", op) and len(args) > 1:
        return _registers(args[1])
    return set()


def hazards_in(text: str) -> list:
    """Loads into LDS in an objdump listing that a vector instruction's scalar result reaches too soon, on any path."""
    found = []
    for body in re.split(r"^[0-9a-f]+ <[^>]+>:\n", text, flags=re.M)[1:]:
        ins, where = [], {}
        for line in body.splitlines():
            m = re.match(r"\s+(\S+)\s*(.*?)\s*//\s*([0-9A-F]+):", line)
            if m:
                where[int(m[3], 16)] = len(ins)
                ins.append((m[1], [a.strip() for a in m[2].split(",")], line))
        before = {i: ([i - 1] if i and ins[i - 1][0] not in ("s_branch", "s_endpgm", "s_setpc_b64") else []) for i in range(len(ins))}
        addresses = sorted(where)
        for i, (op, args, line) in enumerate(ins):
            if op.startswith(("s_branch", "s_cbranch")):
                offset = int(args[-1].split()[0], 0)                       # in words from the next instruction
                target = addresses[i] + 4 + 4 * (offset - 65536 if offset >= 32768 else offset)
                if target in where:
                    before[where[target]].append(i)
        for i, (op, args, line) in enumerate(ins):
            if not (op.startswith("buffer_load") and re.search(r"\blds\b", line)):
                continue
            wanted = set().union(*(_registers(a.split()[0]) for a in args if a))
            todo, seen = [(j, 0) for j in before[i]], {}
            while todo:
                j, states = todo.pop()
                if states >= WAIT_STATES or seen.get(j, WAIT_STATES) <= states:
                    continue
                seen[j] = states
                o, a, text_j = ins[j]
                if _vector_writes(o, a) & wanted:
                    found.append(f"{text_j.strip()}  ->  {line.strip()}  ({states} wait states)")
                    continue
                states += int(a[0], 0) + 1 if o == "s_nop" else 1
                todo += [(k, states) for k in before[j]]
    return found


def lds_load_hazards(path: str) -> list:
    out = []
    for code in code_objects(path):
        if b"gemm_" in code:                      # the kernels with such loads
            out += hazards_in(listing(code))
    return out
