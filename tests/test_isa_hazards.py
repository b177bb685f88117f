"""Static check of this library's own generated gfx950 code for two measured hardware hazards.

On MI355X a ``v_mfma_f32_16x16x16_bf16`` whose accumulator input (SrcC) is the result of a
``v_mfma_f32_16x16x32_bf16`` issued fewer than 5 wait states earlier reads the registers' OLD contents (a probe
with both instructions in one asm block showed it; 5 or more wait states and two products of one shape are fine).
The other order is not safe either: a 16x16x32 product that accumulated onto a 16x16x16 result 4 wait states old,
with no matrix product between the two, came out wrong in its upper two registers in some waves.  The kernels are
written so that no product accumulates onto the result of the other shape at all, at whatever distance (one file
uses one shape only, the others sum each shape in registers of its own), but nothing in the language stops a later
edit or compiler from producing such a pair.  These tests compile the translation units that use both shapes, or
did, to assembly and look for it."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2503_01868_amd", "csrc")
SAFE_WAIT_STATES = 5

MFMA = re.compile(r"^\s*(v_mfma_f32_(\d+x\d+x\d+)\w*)\s+([av])\[(\d+):(\d+)\],\s*([^,]+),\s*([^,]+),\s*(.+?)\s*(?:;.*)?$")
REG = re.compile(r"([av])\[(\d+):(\d+)\]")


def assemble(src, tmp_path):
    hipcc = "/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else shutil.which("hipcc")
    if not hipcc:
        pytest.skip("hipcc not available")
    out = str(tmp_path / (os.path.basename(src) + ".s"))
    cmd = [hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-S", "--cuda-device-only", src, "-o", out]
    proc = subprocess.run(cmd, capture_output=True, text=True)
    assert proc.returncode == 0, proc.stderr[-2000:]
    return open(out).read().splitlines()


def hazards(lines):
    """(line number, text) of every 16x16x16 product that takes a 16x16x32 result as SrcC within the unsafe distance."""
    found = []
    recent = []  # (wait states since issue, register file, lo, hi) of recent 16x16x32 results
    n_mfma = {"16x16x32": 0, "16x16x16": 0}
    for no, line in enumerate(lines, 1):
        text = line.split(";")[0].strip()
        if not text or text.startswith(".") or text.startswith("//"):
            continue
        if text.endswith(":"):  # a label: control flow may join here, forget what was in flight
            recent = []
            continue
        cost = 1
        m_nop = re.match(r"s_nop\s+(\d+)", text)
        if m_nop:
            cost = int(m_nop.group(1)) + 1
        m = MFMA.match(text)
        if m:
            shape = m.group(2)
            if shape in n_mfma:
                n_mfma[shape] += 1
            if shape == "16x16x16":
                c = REG.match(m.group(8).strip())
                if c:
                    for age, rf, lo, hi in recent:
                        if age < SAFE_WAIT_STATES and rf == c.group(1) and not (int(c.group(3)) < lo or int(c.group(2)) > hi):
                            found.append((no, text))
        recent = [(age + cost, rf, lo, hi) for age, rf, lo, hi in recent if age + cost < 16]
        if m and m.group(2) == "16x16x32":
            recent.append((0, m.group(3), int(m.group(4)), int(m.group(5))))
    return found, n_mfma


def test_the_checker_sees_a_planted_pair_and_accepts_a_distant_one():
    bad = ["v_mfma_f32_16x16x32_bf16 v[0:3], v[4:7], v[8:11], v[0:3]", "v_mov_b32 v20, v21",
           "v_mfma_f32_16x16x16_bf16 v[0:3], v[12:13], v[14:15], v[0:3]"]
    assert len(hazards(bad)[0]) == 1
    ok = [bad[0], "s_nop 4", bad[2]]
    assert hazards(ok)[0] == []
    other_regs = [bad[0], "v_mfma_f32_16x16x16_bf16 v[0:3], v[12:13], v[14:15], v[16:19]"]
    assert hazards(other_regs)[0] == []
    reverse = ["v_mfma_f32_16x16x16_bf16 v[0:3], v[12:13], v[14:15], 0", "v_mfma_f32_16x16x32_bf16 v[0:3], v[4:7], v[8:11], v[0:3]"]
    assert hazards(reverse)[0] == []


@pytest.mark.parametrize("unit", ["mr_bwd_kernels.hip", "chain_bwd_kernels.hip"])
def test_no_short_product_accumulates_onto_a_fresh_long_product(unit, tmp_path):
    lines = assemble(os.path.join(CSRC, unit), tmp_path)
    found, n = hazards(lines)
    assert n["16x16x32"] > 0 and n["16x16x16"] > 0, n  # the unit really uses both shapes (else the check is vacuous)
    assert not found, found[:5]


def lone_short_feeds_long(lines):
    """16x16x32 products whose SrcC is the result of a 16x16x16 product issued up to 8 wait states earlier with no other
    matrix product between the two: with 4 such states the upper two registers of the result were wrong in some waves."""
    found, short = [], None  # short: (wait states since issue, register file, lo, hi) of the newest product, if 16x16x16
    for no, line in enumerate(lines, 1):
        text = line.split(";")[0].strip()
        if not text or text.startswith(".") or text.startswith("//"):
            continue
        m = MFMA.match(text)
        if text.endswith(":"):
            short = None
        elif m:
            c = REG.match(m.group(8).strip())
            if m.group(2) == "16x16x32" and c and short and short[1] == c.group(1) \
                    and not (int(c.group(3)) < short[2] or int(c.group(2)) > short[3]) and 2 <= short[0] <= 8:
                found.append((no, text))
            short = (0, m.group(3), int(m.group(4)), int(m.group(5))) if m.group(2) == "16x16x16" else None
        elif short:
            nop = re.match(r"s_nop\s+(\d+)", text)
            short = (short[0] + (int(nop.group(1)) + 1 if nop else 1),) + short[1:]
    return found


def test_the_second_checker_sees_a_planted_pair():
    pair = ["v_mfma_f32_16x16x16_bf16 v[0:3], v[12:13], v[14:15], v[0:3]", "s_nop 3",
            "v_mfma_f32_16x16x32_bf16 v[20:23], v[4:7], v[8:11], v[0:3]"]
    assert len(lone_short_feeds_long(pair)) == 1
    between = pair[:1] + ["v_mfma_f32_16x16x16_bf16 v[16:19], v[12:13], v[14:15], 0"] + pair[1:]
    assert lone_short_feeds_long(between) == []


@pytest.mark.parametrize("unit", ["li_kernels.hip", "mr_bwd_kernels.hip", "chain_bwd_kernels.hip"])
def test_no_long_product_accumulates_onto_a_lone_short_product(unit, tmp_path):
    assert lone_short_feeds_long(assemble(os.path.join(CSRC, unit), tmp_path)) == []


RESULT = re.compile(r"^(\S+)\s+(?:([av])(\d+)|([av])\[(\d+):(\d+)\])(?!\w)")
NO_RESULT = ("global_store", "scratch_store", "buffer_store", "ds_write", "s_")


def mixed_accumulation(lines):
    """(line number, text) of every 16x16x16 or 16x16x32 product whose SrcC was last written by a product of the other one of
    these shapes, in the order of the listing and at any distance; and the number of products of each."""
    found, last, n_mfma = [], {}, {"16x16x32": 0, "16x16x16": 0}  # last: the shape that wrote a register, if a product did
    for no, line in enumerate(lines, 1):
        text = line.split(";")[0].strip()
        if text.startswith(".Lfunc_end"):
            last = {}
        if not text or text.startswith(".") or text.startswith("//"):
            continue
        m, d = MFMA.match(text), RESULT.match(text)
        if m:
            shape, c = m.group(2), REG.match(m.group(8).strip())
            if shape in n_mfma:
                n_mfma[shape] += 1
                if c and any(last.get((c.group(1), r), shape) != shape for r in range(int(c.group(2)), int(c.group(3)) + 1)):
                    found.append((no, text))
            for r in range(int(m.group(4)), int(m.group(5)) + 1):
                last[m.group(3), r] = shape
        elif d and not d.group(1).startswith(NO_RESULT):
            f = d.group(2) or d.group(4)
            for r in range(int(d.group(3) or d.group(5)), int(d.group(3) or d.group(6)) + 1):
                last.pop((f, r), None)
    return found, n_mfma


def test_the_third_checker_sees_planted_pairs_at_any_distance():
    short = "v_mfma_f32_16x16x16_bf16 v[0:3], v[12:13], v[14:15], 0"
    long = "v_mfma_f32_16x16x32_bf16 v[0:3], v[4:7], v[8:11], v[0:3]"
    far = ["s_nop 15", ".LBB0_1:", "v_mfma_f32_16x16x32_bf16 v[20:23], v[4:7], v[8:11], 0"]
    assert len(mixed_accumulation([short] + far + [long])[0]) == 1
    assert len(mixed_accumulation([long] + far + ["v_mfma_f32_16x16x16_bf16 v[0:3], v[12:13], v[14:15], v[0:3]"])[0]) == 1
    assert mixed_accumulation([short, "v_mov_b32 v0, v9", "v_pk_mov_b32 v[1:2], v[9:10], v[9:10]", "ds_read_b32 v3, v9", long])[0] == []
    assert mixed_accumulation([short, ".Lfunc_end0:", long])[0] == []


@pytest.mark.parametrize("unit,short", [("li_kernels.hip", False), ("mr_bwd_kernels.hip", True), ("chain_bwd_kernels.hip", True)])
def test_no_product_accumulates_onto_the_other_shape(unit, short, tmp_path):
    found, n = mixed_accumulation(assemble(os.path.join(CSRC, unit), tmp_path))
    assert n["16x16x32"] > 0 and (n["16x16x16"] > 0) == short, n
    assert not found, found[:5]
