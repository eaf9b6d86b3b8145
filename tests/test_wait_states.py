"""Wait states in the built kernels.  On gfx950 a vector instruction that reads a
scalar register (a lane mask, VCC, a broadcast value) needs two wait states after the
vector instruction that wrote it, and one that reads the result of a
transcendental instruction one.  The compiler puts them there for code it
generates, but not around instructions written in inline assembly, so the machine code of
the library is searched for every such pair."""
import os
import re
import subprocess

import pytest

from paper_2406_16091_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
TRANS = re.compile(r"v_(rcp|rsq|sqrt|exp|log|sin|cos)_")
REG = re.compile(r"\b([sv])(?:(\d+)|\[(\d+):(\d+)\])|\b(vcc)\b")


def _regs(text, kind):
    out = set()
    for m in REG.finditer(text):
        if m.group(5):
            if kind == "s":
                out |= {"vcc"}
        elif m.group(1) == kind:
            lo = int(m.group(2) or m.group(3))
            out |= {(kind, r) for r in range(lo, int(m.group(2) or m.group(4)) + 1)}
    return out


def missing_waits(lines):
    """(line number, text, register) of every read that comes too soon, in a
    disassembly; straight-line distances, forgotten at labels after an
    unconditional jump."""
    found = []
    written = {}  # register -> (wait states needed, time of the write)
    now = 0
    for no, line in enumerate(lines):
        text = line.split("//")[0].strip()
        if not text or text.endswith(":") or not re.match(r"[a-z]", text):
            continue
        op, _, rest = text.partition(" ")
        args = [a.strip() for a in re.split(r",(?![^\[]*\])", rest)]
        if op.startswith("v_"):
            cmp_op = op.startswith("v_cmp")
            carry = re.match(r"v_(add|sub|subrev|addc|subb|subbrev)_co_|v_div_scale|v_mad_[ui]64", op)
            ndst = 2 if carry else 1
            dst, src = " ".join(args[:ndst]), " ".join(args[ndst:])
            if op.startswith(("v_swap", "v_permlane16_swap", "v_permlane32_swap")):
                src = dst = " ".join(args)
            elif re.match(r"v_(fmac|mac|pk_fmac|dot\dc)", op):
                src += " " + args[0]
            reads = _regs(src, "s") | _regs(src, "v")
            if op.startswith("v_div_fmas"):
                reads |= {"vcc"}
            for r in reads:
                need, when = written.get(r, (0, -99))
                if now - when - 1 < need and (need == 2 or not TRANS.match(op)):
                    found.append((no, text, r))
            for r in _regs(dst, "v"):
                written.pop(r, None)
                if TRANS.match(op):
                    written[r] = (1, now)
            if cmp_op or carry or op.startswith(("v_readlane", "v_readfirstlane")):
                for r in _regs(dst, "s"):
                    written[r] = (2, now)
            now += 1
            continue
        if op.startswith("s_"):
            if op == "s_nop":
                now += int(args[0], 0) + 1
                continue
            if op in ("s_branch", "s_endpgm", "s_setpc_b64"):
                written.clear()
            elif not op.startswith(("s_cmp", "s_bitcmp", "s_cbranch", "s_waitcnt", "s_barrier")):
                for r in _regs(args[0], "s"):
                    written.pop(r, None)
        elif op.startswith(("ds_", "global_load", "flat_load", "buffer_load", "scratch_load")):
            for r in _regs(args[0], "v"):
                written.pop(r, None)
        now += 1
    return found


def _disassembly(tmp_path):
    lib = tmp_path / "libpi.so"
    lib.write_bytes(open(build.LIB, "rb").read())
    subprocess.run([OBJDUMP, "--offloading", lib.name], cwd=tmp_path, check=True, capture_output=True)
    for f in sorted(tmp_path.glob(f"libpi.so.*{build.ARCH}")):
        r = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f.name], cwd=tmp_path, check=True,
                           capture_output=True, text=True)
        yield f.name, r.stdout.splitlines()


def test_the_search_finds_and_passes_what_it_should():
    early = ["v_cmp_gt_f32_e64 s[4:5], 0, v1", "v_add_u32_e32 v3, v4, v5", "v_cndmask_b32_e64 v2, v3, v4, s[4:5]"]
    assert {f[2] for f in missing_waits(early)} == {("s", 4), ("s", 5)}
    assert not missing_waits(early[:1] + ["s_nop 1"] + early[2:])
    assert not missing_waits(early[:2] + ["s_and_b64 s[4:5], s[4:5], exec"] + early[2:])
    assert missing_waits(["v_cmp_gt_f32_e32 vcc, 0, v1", "v_cndmask_b32_e32 v2, v3, v4, vcc"])
    assert missing_waits(["v_readlane_b32 s7, v1, 3", "v_add_u32_e32 v3, s7, v5"])
    assert missing_waits(["v_rsq_f32_e32 v1, v2", "v_mul_f32_e32 v3, v1, v5"])
    assert not missing_waits(["v_rsq_f32_e32 v1, v2", "s_nop 0", "v_mul_f32_e32 v3, v1, v5"])


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_the_built_kernels_keep_the_wait_states(tmp_path):
    if not os.path.exists(build.LIB):
        build.build()
    checked = 0
    for name, lines in _disassembly(tmp_path):
        found = missing_waits(lines)
        checked += len(lines)
        assert not found, (name, len(found), found[:8])
    assert checked > 1000
