"""Wait states around inline assembly, on the compiler's listing (no GPU).  The
compiler places the wait states of gfx950 between instructions of its own; it
does not look into an asm block.  Where a block writes or reads a register, the
distances below have to be there all the same:
 * a vector instruction's scalar result (v_readlane, v_readfirstlane, v_cmp)
   read by a vector instruction: two wait states;
 * a vector register just written, read across lanes by DPP: two;
 * the same, read by v_readlane or v_readfirstlane: one."""

import re
import subprocess

import pytest

from paper_2105_11004_amd import build as B

REG = re.compile(r"\b([vs])(\d+)\b|\b([vs])\[(\d+):(\d+)\]")


def _regs(text):
    out = set()
    for a, i, b, lo, hi in REG.findall(text):
        out |= {a + i} if a else {f"{b}{k}" for k in range(int(lo), int(hi) + 1)}
    return out


def missing_waits(listing):
    """(line number, text) of the reads that come too early."""
    bad, recent, in_asm = [], [], False  # recent: (wait states ago, registers written, in an asm block)
    for number, line in enumerate(listing.splitlines(), 1):
        line = line.strip()
        if line.startswith(";;#ASM"):
            in_asm = "START" in line
            continue
        op, _, args = line.split(";")[0].partition(" ")
        if not re.match(r"[vs]_|ds_|global_|buffer_|flat_|scratch_", op):
            continue
        if op == "s_nop":
            recent = [(age + int(args, 0) + 1, w, a) for age, w, a in recent]
            continue
        dest, _, sources = args.partition(",")
        reads, need = _regs(sources), {}
        if op.startswith("v_"):
            need = {r: 2 for r in reads if r[0] == "s"}
            if "_dpp" in op or " row_" in args or "quad_perm" in args:
                # (src0 is the one read across lanes)
                need |= {r: 2 for r in _regs(sources.split(",")[0]) if r[0] == "v"}
            elif op.startswith(("v_readlane", "v_readfirstlane")):
                need |= {r: 1 for r in reads if r[0] == "v"}
        for age, written, asm in recent:
            if (asm or in_asm) and any(age < need.get(r, 0) for r in written):
                bad.append((number, line))
        recent = [(age + 1, w, a) for age, w, a in recent if age < 2]
        if op.startswith("v_"):
            recent.append((0, _regs(dest), in_asm))
    return bad


@pytest.mark.parametrize("source", ["pivchol.hip", "rownorm_csr.hip"])
def test_asm_blocks_keep_their_wait_states(tmp_path, source):
    out = tmp_path / "listing.s"
    subprocess.run([B._hipcc(), "-x", "hip", "-S", "--cuda-device-only", str(B.CSRC / source), "-o", str(out),
                    *B.COMMON_FLAGS], check=True, capture_output=True)
    text = out.read_text()
    assert ";;#ASMSTART" in text
    assert missing_waits(text) == []


def test_scan_sees_a_missing_wait():
    asm = ";;#ASMSTART\n\tv_readlane_b32 s0, v4, 63\n\t;;#ASMEND\n"
    use = "\tv_cmp_eq_u32_e64 s[0:1], s0, v1\n"
    assert missing_waits(asm + "\ts_nop 0\n" + use) != []
    assert missing_waits(asm + "\ts_nop 1\n" + use) == []
    assert missing_waits(asm + "\tv_mov_b32_e32 v9, v8\n\ts_nop 0\n" + use) == []
    dpp = ";;#ASMSTART\n\tv_max_i32_dpp v4, v4, v4 row_shr:1 row_mask:0xf bank_mask:0xf\n\t;;#ASMEND\n"
    assert missing_waits("\tv_mov_b32_e32 v4, v1\n\ts_nop 0\n" + dpp) != []
    assert missing_waits(dpp + "\tv_readlane_b32 s3, v4, 63\n") != []
