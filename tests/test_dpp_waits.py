"""Wait states of the row-broadcast FMAs (v_fmac_f64_dpp in inline asm) in the built device code.

A vector write of a register must lie two wait states before a DPP read of it.  The compiler's hazard handling does not
look into inline asm, so the sources put an s_nop 1 before every straight run of these FMAs.  The check reads the
disassembly of libakra.so and takes every register as just written where a block begins, since what the block before
ends with (register copies, reloads) is the register allocator's choice."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2606_06175_amd", "libakra.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
NEED = 2


def _regs(op):
    m = re.match(r"[-|]*v(?:\[(\d+):(\d+)\]|(\d+)\b)", op)
    if not m:
        return range(0)
    a = int(m.group(1) or m.group(3))
    return range(a, int(m.group(2) or a) + 1)


def _functions(text):
    """(name, [(address, instruction, branch target or None)]) of every function."""
    out = []
    for line in text.splitlines():
        m = re.match(r"^([0-9a-f]+) <(\S+)>:", line)
        if m:
            out.append((m.group(2), int(m.group(1), 16), []))
            continue
        m = re.match(r"^\s+(\S.*?)\s*// ([0-9A-F]+):", line)
        if m and out:
            t = re.search(r"<\S+?\+0x([0-9a-f]+)>\s*$", line) if m.group(1).startswith("s_") else None
            out[-1][2].append((int(m.group(2), 16), m.group(1), out[-1][1] + int(t.group(1), 16) if t else None))
    return [(n, ins) for n, _, ins in out]


def _violations(ins):
    starts = {t for _, _, t in ins if t is not None}
    since = {r: 0 for r in range(512)}  # wait states since the register's last vector write, while below NEED
    seen, bad = 0, []
    for addr, text, target in ins:
        op, _, rest = text.partition(" ")
        ops = [o.strip() for o in rest.split(",")]
        if addr in starts:
            since = {r: 0 for r in range(512)}
        if op.endswith("_f64_dpp"):
            seen += 1
            if any(r in since for r in _regs(ops[1])):
                bad.append("%x %s" % (addr, text))
        n = int(ops[0]) + 1 if op == "s_nop" else 1
        since = {r: w + n for r, w in since.items() if w + n < NEED}
        if op.startswith("v_") and not op.startswith("v_cmp"):
            for o in ops[:2 if "swap" in op else 1]:
                since.update((r, 0) for r in _regs(o))
        if op == "s_branch" or op.startswith("s_cbranch"):
            since = {r: 0 for r in range(512)}
    return seen, bad


def test_row_broadcast_waits(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    assert os.path.exists(LIB), "build libakra.so first"
    shutil.copy(LIB, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    total, bad = 0, []
    for f in sorted(os.listdir(tmp_path)):
        if not f.endswith("gfx950"):
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f], cwd=tmp_path, check=True, capture_output=True,
                              text=True).stdout
        if "_f64_dpp" not in text:
            continue
        for name, ins in _functions(text):
            if any("_f64_dpp" in t for _, t, _ in ins):
                n, b = _violations(ins)
                total += n
                bad += ["%s %s" % (name, v) for v in b]
    assert total > 1000  # the synthesis and the batched adjoint are there
    assert not bad, bad[:5]
