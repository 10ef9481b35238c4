"""What the compiler does not check of the hand-written loads into LDS and matrix products (csrc/gemm_tile.hpp), looked up in
the gfx950 code of a built library.

Hazards inside inline assembly are the author's.  A buffer load must not read a scalar register within five wait states
after a vector instruction wrote it (a lane read, a compare, a carry), nor go by m0 in the instruction after the one that
writes it.  The kernels' descriptors are made by scalar
instructions, which the hardware waits for.  A matrix product must not read a register within two wait states after a vector
instruction wrote it, and its result is read by others 18 wait states later at the earliest (more than the largest product
takes).  Whether all that holds depends on what the compiler does with the code
around, copies of a sum among it, so every build looks.
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
TO_PRODUCT, FROM_PRODUCT = 2, 18
BY_COMPILER = ("gemm_slim_kernel", "gemm_f32_")   # kernels whose products are builtins: the compiler keeps the hardware's own, shorter, states
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


def _functions(text: str, wanted=lambda name, body: True):
    """Name, instructions (mnemonic, operands, line) and, for each, those that can run right before it, of a listing's functions."""
    parts = re.split(r"^[0-9a-f]+ <([^>]+)>:\n", text, flags=re.M)
    for name, body in zip(parts[1::2], parts[2::2]):
        if not wanted(name, body):
            continue
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
        yield name, ins, before


def _within(ins, before, i, limit, hit):
    """Instructions that hit() accepts less than `limit` wait states ahead of instruction i, on any path, with the states between."""
    todo, seen = [(j, 0) for j in before[i]], {}
    while todo:
        j, states = todo.pop()
        if states >= limit or seen.get(j, limit) <= states:
            continue
        seen[j] = states
        if hit(j):
            yield f"{ins[j][2].strip()}  ->  {ins[i][2].strip()}  ({states} wait states)"
            continue
        states += int(ins[j][1][0], 0) + 1 if ins[j][0] == "s_nop" else 1
        todo += [(k, states) for k in before[j]]


def hazards_in(text: str) -> list:
    """Loads into LDS in an objdump listing that a vector instruction's scalar result, or m0, reaches too soon, on any path."""
    found = []
    for _, ins, before in _functions(text, lambda name, body: re.search(r"\blds\b", body)):
        for i, (op, args, line) in enumerate(ins):
            if not (op.startswith("buffer_load") and re.search(r"\blds\b", line)):
                continue
            wanted = set().union(*(_registers(a.split()[0]) for a in args if a))
            found += _within(ins, before, i, WAIT_STATES, lambda j: _vector_writes(ins[j][0], ins[j][1]) & wanted)
            found += _within(ins, before, i, 1, lambda j: ins[j][0].startswith("s_") and ins[j][1][0] == "m0")
    return found


def _lanes(operand: str) -> set:
    m = re.match(r"([av])(\d+)$", operand) or re.match(r"([av])\[(\d+):(\d+)\]", operand)
    return {(m[1], r) for r in range(int(m[2]), int(m[m.lastindex]) + 1)} if m else set()


def product_hazards_in(text: str, but: tuple = ()) -> list:
    """Matrix products in an objdump listing (functions whose name contains none of `but`) that read a vector instruction's result, or
    whose own result another instruction reads or overwrites, too soon, on any path."""
    found = []
    for _, ins, before in _functions(text, lambda name, body: "v_mfma" in body and not any(family in name for family in but)):
        regs = [[_lanes(a) for a in args] for _, args, _ in ins]
        product = [op.startswith("v_mfma") for op, _, _ in ins]
        # a swap writes both its operands
        writes = [r[0] | (r[1] if "swap" in ins[i][0] and len(r) > 1 else set()) if r and ins[i][0].startswith("v_") else set()
                  for i, r in enumerate(regs)]
        for i in range(len(ins)):
            touched = set().union(*regs[i])
            if product[i]:
                found += _within(ins, before, i, TO_PRODUCT, lambda j: not product[j] and writes[j] & touched)
            elif touched:
                found += _within(ins, before, i, FROM_PRODUCT, lambda j: product[j] and writes[j] & touched)
    return found


def hazards(path: str) -> list:
    """Both kinds in a built library.  Products are looked at in every kernel but those that leave them to the compiler, so that no kernel
    that comes to write them out can be forgotten."""
    out = []
    for code in code_objects(path):
        text = listing(code)
        out += hazards_in(text) + product_hazards_in(text, BY_COMPILER)
    return out
