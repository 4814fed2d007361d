"""The built kernels, in the AMD assembly: no work-group barrier may be reached
with a write to LDS still on its way (the value a wave reads after the barrier
could then be the one before the write)."""
import os
import re
import struct
import subprocess

import pytest

OBJDUMP = "/opt/rocm/lib/llvm/bin/llvm-objdump"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
WRITES = re.compile(r"ds_(?!read|load|bpermute|permute|swizzle|nop|consume|append)")


def pending_writes(lines):
    """functions and offsets of the barriers that a wave can reach with LDS
    writes pending, and the number of barriers, in a disassembly"""
    bad, barriers = [], 0
    for name, ins in _functions(lines):
        if not any(op == "s_barrier" for _, op, _ in ins):
            continue
        at = {a: i for i, (a, _, _) in enumerate(ins)}
        state = [None] * len(ins)       # pending on entry: None = not reached
        work = [(0, False)]
        while work:
            i, p = work.pop()
            while i < len(ins) and (state[i] is None or (p and not state[i])):
                state[i] = bool(state[i]) or p
                _, op, arg = ins[i]
                if WRITES.match(op):
                    p = True
                elif op == "s_waitcnt" and ("lgkmcnt(0)" in arg or arg.strip() == "0"):
                    p = False
                elif op in ("s_endpgm", "s_setpc_b64"):
                    break
                elif op == "s_branch" or op.startswith("s_cbranch"):
                    to = at[int(re.search(r"\+0x([0-9a-f]+)>", arg).group(1), 16)] if "+0x" in arg else 0
                    work.append((to, p))
                    if op == "s_branch":
                        break
                i += 1
        for (a, op, _), p in zip(ins, state):
            if op == "s_barrier":
                barriers += 1
                if p:
                    bad.append((name, hex(a)))
    return bad, barriers


def _functions(lines):
    """(name, [(offset, instruction, operands)]) of each function of a disassembly"""
    name, base, ins = None, 0, []
    for line in lines:
        m = re.match(r"^([0-9a-f]+) <(\S+)>:", line)
        if m:
            if name and ins:
                yield name, ins
            base, name, ins = int(m.group(1), 16), m.group(2), []
            continue
        m = re.match(r"^\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+): [0-9A-F ]+(<.*>)?", line)
        if m and name:
            ins.append((int(m.group(3), 16) - base, m.group(1), m.group(2) + " " + (m.group(4) or "")))
    if name and ins:
        yield name, ins


def _code_objects(path):
    """the gfx950 code objects of a built library, one per source"""
    data = open(path, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, tl = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + tl] and size:
                yield data[at + off:at + off + size]
            p += 24 + tl
        at = data.find(MAGIC, p)


def test_scan_finds_a_barrier_without_its_wait():
    """a loop whose barrier stands at its head: the wait before the loop does not cover the write at its end"""
    asm = """0000000000000100 <k>:
	ds_write_b64 v0, v[1:2]      // 000000000100: D89A0000
	s_waitcnt lgkmcnt(0)         // 000000000104: BF8CC07F
	s_barrier                    // 000000000108: BF8A0000
	ds_write_b64 v0, v[1:2]      // 00000000010C: D89A0000
	s_cbranch_scc1 65532         // 000000000110: BF85FFFC <k+0x8>
	s_endpgm                     // 000000000114: BF810000
""".splitlines()
    assert pending_writes(asm) == ([("k", "0x8")], 1)
    fixed = [l.replace("s_waitcnt lgkmcnt(0)         // 000000000104", "s_nop 0 // 000000000104") for l in asm]
    fixed.insert(3, "	s_waitcnt lgkmcnt(0)         // 000000000106: BF8CC07F")
    assert pending_writes([l.replace("<k+0x8>", "<k+0x6>") for l in fixed]) == ([], 1)


def test_no_barrier_with_lds_writes_pending(tmp_path):
    from paper_2305_17341_amd import he
    if not os.path.exists(he.LIB_PATH) or not os.path.exists(OBJDUMP):
        pytest.skip("library or disassembler not there")
    total = 0
    for k, code in enumerate(_code_objects(he.LIB_PATH)):
        f = tmp_path / f"{k}.co"
        f.write_bytes(code)
        r = subprocess.run([OBJDUMP, "-d", str(f)], capture_output=True, text=True, check=True)
        bad, n = pending_writes(r.stdout.splitlines())
        total += n
        assert not bad
    assert total > 0
