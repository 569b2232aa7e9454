"""The main loops' MFMAs and LDS reads are written out as instructions, so the compiler neither waits for the ones nor keeps
its distance from the others: what it places between them is checked here, in the code that was built.  In every block that
holds MFMAs: no register of an LDS read is touched before the read has been waited for, operands of an MFMA come from an LDS
read and nowhere else (a copy in between would need wait states), and nothing but an MFMA touches an accumulator within the
18 wait states an MFMA may take."""
import os
import re
import subprocess

import pytest

from paper_2406_06858_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
MFMA_WAIT_STATES = 18
_REG = re.compile(r"\b([va])(?:(\d+)|\[(\d+):(\d+)\])")


def _regs(text):
    out = set()
    for kind, one, lo, hi in _REG.findall(text):
        out.update((kind, r) for r in (range(int(lo), int(hi) + 1) if lo else (int(one),)))
    return out


def _check_block(lines):
    """First violation among the instructions of one block, or None."""
    pending = []                      # registers of LDS reads that may still be on their way, oldest first
    since = {}                        # accumulator -> wait states since an MFMA wrote it
    copied = set()                    # registers last written by something other than an LDS read
    for line in lines:
        op, _, rest = line.partition(" ")
        args = rest.split(",")
        if op == "s_waitcnt":
            m = re.search(r"lgkmcnt\((\d+)\)", rest)
            if m:
                pending = pending[len(pending) - int(m[1]):] if int(m[1]) else []
            states = 1
        else:
            states = int(rest.strip(), 0) + 1 if op == "s_nop" else 1
            touched = _regs(rest)
            for p in pending:
                if p & touched:
                    return f"{line}: a register of an LDS read before its wait"
            dst = _regs(args[0]) if op.startswith(("v_", "ds_read", "buffer_load", "global_load")) and " lds" not in rest else set()
            if op.startswith("v_mfma"):
                if (_regs(args[1]) | _regs(args[2])) & copied:
                    return f"{line}: an operand that is no LDS read's"
            else:
                near = [r for r in touched if since.get(r, 99) < MFMA_WAIT_STATES]
                if near:
                    return f"{line}: {near[0]} right behind an MFMA"
                if op.startswith("ds_read"):
                    pending.append(dst)
                    copied -= dst
                else:
                    copied |= dst
            for r in since:
                since[r] += states
            if op.startswith("v_mfma"):
                since.update((r, 0) for r in dst)
    return None


def _blocks(text):
    block = []
    for line in text.splitlines():
        line = line.split("//")[0].strip()
        if not line or line.endswith(":"):
            if block:
                yield block
            block = []
            continue
        block.append(line)
        if line.startswith(("s_cbranch", "s_branch", "s_endpgm")):
            yield block
            block = []
    if block:
        yield block


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_nothing_between_the_written_out_instructions(tmp_path):
    lib = tmp_path / "lib.so"
    lib.symlink_to(build.LIB)
    subprocess.run([OBJDUMP, "--offloading", str(lib)], cwd=tmp_path, check=True, capture_output=True)
    objects = [p for p in tmp_path.iterdir() if "gfx950" in p.name]
    assert objects
    with_mfma = 0
    for o in objects:
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", str(o)], check=True, capture_output=True, text=True).stdout
        for block in _blocks(text):
            if any(i.startswith("v_mfma") for i in block):
                with_mfma += 1
                assert _check_block(block) is None
    assert with_mfma >= 10 * build.N_CFGS


@pytest.mark.parametrize("lines,what", [
    (["ds_read_b64_tr_b16 v[2:3], v9", "v_mov_b32_e32 v4, v2", "s_waitcnt lgkmcnt(0)"], "before its wait"),
    (["ds_read_b128 v[0:3], v9", "v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]"], "before its wait"),
    (["ds_read_b128 v[0:3], v9", "s_waitcnt lgkmcnt(0)", "v_mov_b32_e32 v4, v0", "v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]"], "no LDS read's"),
    (["v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]", "s_nop 7", "v_accvgpr_read_b32 v9, a2"], "right behind"),
    (["v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]", "s_nop 15", "s_nop 15", "v_accvgpr_read_b32 v9, a2"], None),
    (["ds_read_b128 v[0:3], v9", "ds_read_b128 v[4:7], v9", "s_waitcnt lgkmcnt(1)", "v_mov_b32_e32 v8, v0"], None),
])
def test_the_check_finds_what_it_looks_for(lines, what):
    got = _check_block(lines)
    assert got is None if what is None else what in got
