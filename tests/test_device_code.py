"""The built device code, read back: no data register of a store in flight is overwritten.

A vector store of more than 8 bytes a lane reads its data registers after it has issued; a vector
instruction that writes one of them needs two wait states in between.  The compiler inserts them,
but not behind a buffer store whose offset is in a scalar register, and there the hardware needs
them too (partial sums of 64-row tiles were stored with the next block's first value in a quarter
of the lanes)."""
import os
import re
import shutil
import subprocess

import pytest

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
WIDE_STORE = re.compile(r"(buffer|global|flat|scratch)_store_(dwordx[34]|format_xyz|format_xyzw)$")
WAIT_STATES = 2


def _registers(operand):
    m = re.match(r"([va])\[(\d+):(\d+)\]$", operand) or re.match(r"([va])(\d+)()$", operand)
    if not m:
        return set()
    return {(m.group(1), r) for r in range(int(m.group(2)), int(m.group(3) or m.group(2)) + 1)}


def parse(lines):
    """(function, address, opcode, operands, branch target or None) of a disassembly's lines."""
    base, fn, out = 0, None, []
    for ln in lines:
        m = re.match(r"([0-9a-f]+) <(.+)>:", ln)
        if m:
            base, fn = int(m.group(1), 16), m.group(2)
            continue
        m = re.match(r"\s+(\S+)(.*?)//\s*([0-9A-F]+):", ln)
        if not m:
            continue
        target = re.search(r"<%s\+0x([0-9a-f]+)>" % re.escape(fn), ln) if "branch" in m.group(1) else None
        out.append((fn, int(m.group(3), 16), m.group(1), [x.strip() for x in m.group(2).split(",")],
                    base + int(target.group(1), 16) if target else None))
    return out


def overwritten_stores(code):
    at = {c[1]: i for i, c in enumerate(code)}
    found = []
    for i, (fn, _, op, args, _) in enumerate(code):
        if not WIDE_STORE.match(op):
            continue
        data = _registers(args[0] if op.startswith("buffer") else args[1])
        todo, seen = [(i + 1, 0)], set()
        while todo:
            j, waited = todo.pop()
            if waited >= WAIT_STATES or j >= len(code) or code[j][0] != fn or (j, waited) in seen:
                continue
            seen.add((j, waited))
            _, _, op2, args2, target = code[j]
            if op2 == "s_endpgm":
                continue
            if op2.startswith("v_") and _registers(args2[0]) & data:
                found.append("%s: %s %s, then %s %s" % (fn, op, ", ".join(args), op2, ", ".join(args2)))
                continue
            waited += 1 + (int(args2[0], 0) if op2 == "s_nop" else 0)
            if target is not None:
                todo.append((at[target], waited))
            if op2 != "s_branch":
                todo.append((j + 1, waited))
    return found


def test_the_reader_sees_an_overwritten_store():
    text = """
0000000000000100 <k>:
	buffer_store_dwordx4 v[50:53], v58, s[4:7], s0 offen       // 000000000100: E07C1000
	s_cbranch_scc0 2                                           // 000000000108: BF840002 <k+0x14>
	v_mov_b32_e32 v1, v2                                       // 00000000010C: 7E020302
	v_cvt_i32_f32_e32 v53, v3                                  // 000000000110: 7E6A1103
	%s// 000000000114: 7E641122
	s_endpgm                                                   // 000000000118: BF810000
"""
    assert len(overwritten_stores(parse((text % "v_cvt_i32_f32_e32 v50, v34 ").split("\n")))) == 1   # by the branch
    assert not overwritten_stores(parse((text % "v_cvt_i32_f32_e32 v54, v34 ").split("\n")))
    assert not overwritten_stores(parse((text % "v_cvt_i32_f32_e32 v50, v34 ").replace("s_cbranch_scc0 2",
                                                                                     "s_nop 1").split("\n")))


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="llvm-objdump not installed")
def test_no_store_data_overwritten(tmp_path):
    import paper_2609_32922_amd._lib as L
    if not os.path.exists(L.LIB_PATH):
        from paper_2609_32922_amd import build
        build.build()
    lib = shutil.copy(L.LIB_PATH, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=tmp_path, capture_output=True, check=True)
    objects = sorted(f for f in os.listdir(tmp_path) if f.endswith("gfx950"))
    assert objects
    stores, found = 0, []
    for f in objects:
        r = subprocess.run([OBJDUMP, "-d", os.path.join(tmp_path, f)], capture_output=True, text=True, check=True)
        code = parse(r.stdout.split("\n"))
        stores += sum(1 for c in code if WIDE_STORE.match(c[2]))
        found += overwritten_stores(code)
    assert stores > 100          # (the reader still finds the stores)
    assert not found, "\n".join(found)
