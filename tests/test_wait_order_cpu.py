"""The library's own gfx950 code, disassembled: matrix instructions written as asm are hidden from the compiler's hazard
recogniser, and where the column sums wait for their results (three s_nop 15 in a row) no instruction that touches a result may
come ahead of the wait.  The results of the last four matrix instructions on every path to the wait count: an older one has long
been written."""

import os
import re
import shutil
import subprocess

import pytest

from paper_2406_12018_amd import build

OBJDUMP = next((p for p in ("/opt/rocm/llvm/bin/llvm-objdump", shutil.which("llvm-objdump")) if p and os.path.exists(p)), None)


def registers(operand):
    m = re.fullmatch(r"v(\d+)|v\[(\d+):(\d+)\]", operand)
    if not m:
        return set()
    return {int(m[1])} if m[1] else set(range(int(m[2]), int(m[3]) + 1))


def functions(text):
    """name, [(address, mnemonic, operands, branch target)]"""
    name, code = None, []
    for line in text.splitlines():
        m = re.match(r"[0-9a-f]+ <(\S+)>:", line)
        if m:
            if name:
                yield name, code
            name, code = m[1], []
            continue
        m = re.match(r"\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+):.*?(?:<\S+\+0x([0-9a-f]+)>)?$", line)
        if m:
            code.append((int(m[3], 16), m[1], [x.strip() for x in m[2].split(",")], m[4] and int(m[4], 16)))
    if name:
        yield name, code


def waits_out_of_order(code):
    """Positions of waits that an instruction which touches a waited-for result precedes, and the number of waits."""
    start, at = code[0][0], {c[0]: i for i, c in enumerate(code)}
    came_from = {}  # position -> positions that may precede it
    for i, (_, op, _, target) in enumerate(code):
        if i + 1 < len(code) and op not in ("s_branch", "s_endpgm"):
            came_from.setdefault(i + 1, []).append(i)
        if op.startswith(("s_branch", "s_cbranch")):
            came_from.setdefault(at[start + target], []).append(i)

    is_wait = lambda i: i + 2 < len(code) and all(code[i + x][1] == "s_nop" and code[i + x][2] == ["15"] for x in range(3))
    bad, waits = [], 0
    for i in range(len(code)):
        if not is_wait(i):
            continue
        waits += 1
        touched, work, seen = [], [(p, 0, frozenset()) for p in came_from.get(i, [])], set()
        while work:
            p, found, after = work.pop()  # after: registers touched between p and the wait
            _, op, operands, _ = code[p]
            if op.startswith("v_mfma"):
                if registers(operands[0]) & after:
                    touched.append(p)
                found += 1  # its own operands are the matrix pipe's business
            elif op.startswith(("v_", "ds_", "global_", "buffer_")):
                for x in operands:
                    after = after | registers(x)
            if found == 4 or op == "s_nop" and operands == ["15"] or (p, found) in seen:
                continue
            if len(came_from.get(p, [])) > 1 or (p - 1) not in came_from.get(p, []):
                seen.add((p, found))
            work += [(x, found, after) for x in came_from.get(p, [])]
        if touched:
            bad.append((i, code[i][0]))
    return bad, waits


@pytest.mark.skipif(OBJDUMP is None, reason="no llvm-objdump")
def test_nothing_touches_a_matrix_result_ahead_of_its_wait(tmp_path):
    if not os.path.exists(build.LIB_PATH):
        build.build()
    shutil.copy(build.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, stdout=subprocess.DEVNULL)
    waits, bad = {}, []
    for f in sorted(tmp_path.glob("lib.so.*gfx950")):
        text = subprocess.run([OBJDUMP, "-d", str(f)], check=True, stdout=subprocess.PIPE, text=True).stdout
        for name, code in functions(text) if "colsum_mfma_kernel" in text else ():
            if "colsum_mfma_kernel" in name:
                out_of_order, waits[name] = waits_out_of_order(code)
                bad += [(name, hex(a)) for _, a in out_of_order]
    assert len(waits) == 4 and min(waits.values()) >= 3, waits  # two head dimensions, blocks of 128 and of 256 keys
    assert not bad, bad
