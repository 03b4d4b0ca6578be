"""The built kernels' machine code: no vector register or spill slot is written
between the start of a block where divergent lanes meet again and the
instruction that restores their execution mask.  The compiler puts such a copy or
spill there when the saved mask itself has been spilled; the lanes that did not
take the branch then keep whatever the register or slot held (wrong values, and
wild addresses where the value was an index)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2202_02319_amd import _lib

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
EXEC_WRITE = re.compile(r"s_\w+ exec|s_\w*saveexec")
RESTORE = re.compile(r"s_or_b64 exec, exec")
# vector instructions that write no lane's register or slot by the execution mask
OTHER = ("v_writelane", "v_readlane", "v_readfirstlane", "v_cmp", "v_nop")
WRITES = re.compile(r"v_|ds_read|ds_bpermute|global_load|flat_load|scratch_")


def _kernels(lib, tmp):
    so = shutil.copy(lib, tmp)
    subprocess.run([OBJDUMP, "--offloading", so], check=True, capture_output=True, cwd=tmp)
    for f in sorted(os.listdir(tmp)):
        if not f.endswith("gfx950"):
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", os.path.join(tmp, f)], check=True,
                              capture_output=True, text=True).stdout
        for part in re.split(r"\n(?=[0-9a-f]+ <)", text):
            m = re.match(r"([0-9a-f]+) <(\w+)>:\n", part)
            if m:
                yield m.group(2), int(m.group(1), 16), part


def _misplaced(start, part):
    """Writes ahead of the restore, with the number of join blocks (the targets of branches over a masked region)."""
    ins, where = [], {}
    for m in re.finditer(r"^\t(\S.*?)\s*// ([0-9A-F]+):[0-9A-F ]*(?:<\w+\+0x([0-9a-f]+)>)?", part, re.M):
        where[int(m.group(2), 16)] = len(ins)
        ins.append((m.group(1), m.group(3)))
    out = []
    targets = {where[start + int(t, 16)] for op, t in ins if t}
    joins = {where[start + int(t, 16)] for op, t in ins if op.startswith("s_cbranch_execz") and t}
    for k in joins:
        writes = []
        for i in range(k, len(ins)):
            op = ins[i][0]
            if i > k and i in targets:   # the next block
                break
            if RESTORE.match(op):
                out += writes
            if EXEC_WRITE.match(op) or op.startswith(("s_branch", "s_cbranch", "s_endpgm")):
                break
            if WRITES.match(op) and not op.startswith(OTHER):
                writes.append(op)
    return len(joins), out


def test_no_write_before_the_mask_is_restored(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip(f"{OBJDUMP} is missing")
    seen, joins, bad = 0, 0, {}
    for name, start, part in _kernels(_lib.LIB_PATH, tmp_path):
        seen += 1
        n, found = _misplaced(start, part)
        joins += n
        if found:
            bad[name] = found
    assert seen > 100 and joins > 1000
    assert not bad
