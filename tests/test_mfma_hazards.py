"""Compiled kernels: distances between matrix-core products and what reads them.

The compiler puts no wait states between a 16x16x32 and a 16x16x16 bf16 product
that accumulate on the same registers, in either order, and the card then
returns wrong values (a K16 step right after a K32 step: wrong rows 0 and 1 of
every quad; a K32 step right after a K16 step: rows 2 and 3; every time).  A
product's result may be read after 8 wait states, which is what the compiler
leaves before every other reader.  So no such pair may lie closer than that in
the library, along any path of the code, branches included.

The scan follows the disassembly of the library built from this repository.
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2606_27229_amd import carve

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
WAIT = 8
PRODUCTS = ("v_mfma_f32_16x16x16_bf16", "v_mfma_f32_16x16x32_bf16")
_REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")


def _regs(operand):
    m = _REG.search(operand)
    if not m:
        return frozenset()
    lo, hi = (int(m.group(2)), int(m.group(3))) if m.group(2) else (int(m.group(4)),) * 2
    return frozenset((m.group(1), i) for i in range(lo, hi + 1))


def _listing(text):
    """[(address within the code, mnemonic, operands, branch target)] per function."""
    fn, base, out = None, 0, {}
    for line in text.splitlines():
        m = re.match(r"^([0-9a-f]+) <(.+)>:$", line)
        if m:
            base, fn = int(m.group(1), 16), m.group(2)
            out[fn] = []
            continue
        m = re.match(r"^\s+(\S+)\s*(.*?)\s*//\s*([0-9A-Fa-f]+):(.*)$", line)
        if not m or fn is None:
            continue
        t = re.search(r"<[^>]*?(?:\+0x([0-9a-f]+))?>\s*$", m.group(4))
        target = base + int(t.group(1) or "0", 16) if t else None
        out[fn].append((int(m.group(3), 16), m.group(1), [o.strip() for o in m.group(2).split(",")], target))
    return out


def close_pairs(text):
    """(function, first address, second address, wait states) of every K16 / K32
    pair on one accumulator, and of every other access to a product's result,
    closer than WAIT."""
    bad = []
    for fn, ins in _listing(text).items():
        at = {x[0]: i for i, x in enumerate(ins)}
        for i, (addr, op, args, _) in enumerate(ins):
            if op not in PRODUCTS:
                continue
            dst = _regs(args[0])
            work, seen = [(i + 1, 0)], {}
            while work:
                j, d = work.pop()
                while j < len(ins) and d < WAIT and seen.get(j, WAIT) > d:
                    seen[j] = d
                    addr2, op2, args2, target = ins[j]
                    if op2 == "s_endpgm":
                        break
                    if op2 == "s_nop":
                        d, j = d + int(args2[0], 0) + 1, j + 1
                        continue
                    touched = [k for k, o in enumerate(args2) if _regs(o) & dst]
                    if touched:
                        # a product of the same kind accumulating on (or merely
                        # overwriting) the result is interlocked
                        chained = op2 == op and all(k in (0, 3) for k in touched)
                        if not chained:
                            bad.append((fn, hex(addr), hex(addr2), d))
                        break
                    if op2 == "s_branch":
                        j, d = at[target], d + 1
                        continue
                    if op2.startswith("s_cbranch"):
                        work.append((at[target], d + 1))
                    d, j = d + 1, j + 1
    return bad


def _text(*lines):
    out = ["0000000000001000 <f>:"]
    for i, (ins, target) in enumerate(lines):
        out.append("\t%s // %012X: 00000000%s" % (ins, 0x1000 + 4 * i, "" if target is None else " <f+0x%x>" % (4 * target)))
    return "\n".join(out)


K32 = ("v_mfma_f32_16x16x32_bf16 v[4:7], v[8:11], v[12:15], 0", None)
K16 = ("v_mfma_f32_16x16x16_bf16 v[0:3], v[8:9], v[12:13], v[4:7]", None)
END = ("s_endpgm", None)


def test_scan_on_short_listings():
    assert close_pairs(_text(K32, K16, END))
    assert close_pairs(_text(K32, ("s_nop 6", None), K16, END))
    assert not close_pairs(_text(K32, ("s_nop 7", None), K16, END))
    # along a taken branch, past a product that has nothing to do with it
    assert close_pairs(_text(K32, ("s_cbranch_scc0 2", 4), ("s_nop 7", None), END,
                             ("v_mfma_f32_16x16x32_bf16 v[20:23], v[8:11], v[12:15], 0", None), K16, END))
    # the same kind chained, and an ordinary reader
    assert not close_pairs(_text(K32, ("v_mfma_f32_16x16x32_bf16 v[4:7], v[8:11], v[12:15], v[4:7]", None),
                                 ("s_nop 7", None), END))
    assert close_pairs(_text(K32, ("v_add_f32_e32 v5, v4, v5", None), END))


def test_library_keeps_its_distances(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("llvm-objdump is not installed")
    carve.load_library()
    lib = shutil.copy(carve.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", str(lib)], cwd=tmp_path, check=True, capture_output=True)
    objs = sorted(p for p in os.listdir(tmp_path) if p.endswith("gfx950"))
    assert objs
    nprod, bad = 0, []
    for o in objs:
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(tmp_path / o)], check=True, capture_output=True,
                              text=True).stdout
        nprod += sum(text.count(p) for p in PRODUCTS)
        bad += close_pairs(text)
    assert nprod > 10000   # (the listing was read)
    assert not bad, bad[:10]
