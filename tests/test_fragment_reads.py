"""The matrix fragments' LDS reads in the built library: nothing touches a register in flight.

The token loops read their fragments by inline assembly, so that the compiler does not hold them
back behind the LDS DMA, and wait for them in a later statement.  To the compiler such a read has
delivered at once: were it to copy, spill or reuse a destination before the wait, the kernel would
work on what was there before, or the read would land on something else.  This follows every path
through the disassembly of each kernel and checks that between an LDS read and the wait that
covers it no instruction reads or writes the read's destination.  (LDS operations of a wave return
in order; lgkmcnt counts the ones outstanding.)
"""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2606_22932_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
LGKM = re.compile(r"ds_|s_load|s_buffer_load|s_memtime|s_memrealtime|s_sendmsg")


def code_objects(path):
    """The gfx950 code objects bundled in a shared library."""
    data = open(path, "rb").read()
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        at = m.start() + 24
        (n,), at = struct.unpack_from("<Q", data, at), at + 8
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, at)
            name = data[at + 24:at + 24 + length]
            at += 24 + length
            if b"gfx950" in name and size:
                yield data[m.start() + off:m.start() + off + size]


def kernels(listing):
    """(name, [(address, op, operands)]) of each function of a disassembly."""
    name, ins = None, []
    for line in listing.splitlines():
        head = re.match(r"[0-9a-f]+ <(\w+)>:", line)
        if head:
            if ins:
                yield name, ins
            name, ins = head.group(1), []
            continue
        code, _, tail = line.partition("//")
        if tail and code.strip():
            op, _, rest = code.strip().partition(" ")
            ins.append((int(tail.split(":")[0], 16), op, rest))
    if ins:
        yield name, ins


def registers(text):
    out = set()
    for a, b, c in re.findall(r"\bv\[(\d+):(\d+)\]|\bv(\d+)\b", text):
        out.update([int(c)] if c else range(int(a), int(b) + 1))
    return out


def touched_in_flight(ins):
    """Instructions that read or write the destination of an LDS read in flight."""
    index = {addr: i for i, (addr, _, _) in enumerate(ins)}
    jump = {}
    for i, (addr, op, rest) in enumerate(ins):
        if op == "s_branch" or op.startswith("s_cbranch"):
            k = int(rest.split()[0])
            jump[i] = index[addr + 4 + 4 * (k - 65536 if k >= 32768 else k)]
    regs = [registers(rest) for _, _, rest in ins]
    targets, seen, bad = set(jump.values()), set(), []
    work = [(0, ())]                        # (instruction, destinations in flight, oldest first)
    while work:
        i, flight = work.pop()
        while i < len(ins):
            if i in targets:
                if (i, flight) in seen:
                    break
                seen.add((i, flight))
            addr, op, rest = ins[i]
            if op == "s_waitcnt":
                left = re.search(r"lgkmcnt\((\d+)\)", rest)
                left = int(left.group(1)) if left else (0 if rest.strip() == "0" else len(flight))
                flight = flight[max(0, len(flight) - left):]
            else:
                if any(regs[i] & set(d) for d in flight):
                    bad.append("%x %s %s" % (addr, op, rest))
                if op.startswith("ds_read"):
                    flight += (tuple(sorted(registers(rest.split(",")[0]))),)
                elif LGKM.match(op):
                    flight += ((),)
            while flight and not flight[0]:
                flight = flight[1:]
            if op == "s_endpgm":
                break
            if op == "s_branch":
                i = jump[i]
                continue
            if i in jump:
                work.append((jump[i], flight))
            i += 1
    return bad


def test_checker_sees_a_read_without_its_wait():
    ins = [(0, "ds_read_b64_tr_b16", "v[2:3], v9"), (8, "ds_read_b64_tr_b16", "v[4:5], v9"),
           (16, "s_waitcnt", "lgkmcnt(1)"), (20, "v_mov_b32_e32", "v7, v2"), (24, "s_cbranch_scc1", "1"),
           (28, "s_waitcnt", "lgkmcnt(0)"), (32, "v_mov_b32_e32", "v8, v5"), (36, "s_endpgm", "")]
    assert touched_in_flight(ins) == ["20 v_mov_b32_e32 v8, v5"]     # by the branch only
    assert touched_in_flight(ins[:4] + ins[5:]) == []


@pytest.mark.skipif(shutil.which(OBJDUMP) is None or not os.path.exists(build.LIB),
                    reason="needs llvm-objdump and the library")
def test_no_instruction_touches_a_fragment_in_flight(tmp_path):
    found = 0
    for n, obj in enumerate(code_objects(build.LIB)):
        path = tmp_path / ("%d.o" % n)
        path.write_bytes(obj)
        listing = subprocess.run([OBJDUMP, "-d", str(path)], capture_output=True, text=True, check=True).stdout
        for name, ins in kernels(listing):
            if any(op == "ds_read_b64_tr_b16" for _, op, _ in ins):
                found += 1
                assert touched_in_flight(ins) == [], name
    assert found > 50
