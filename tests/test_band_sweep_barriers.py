"""Barriers of the sweep by layers, in the assembly of the kernels as they are built: a wave that goes through one has waited for all
its LDS operations, or says what it has waited for instead."""
import os
import re
import subprocess

from paper_1707_08265_amd import build as lib_build


def barriers(asm, kernel):
    """What stands in front of every barrier of the kernel, in its basic block, the nearest instruction first."""
    lines = asm[re.search(rf"^\w*{kernel}\w*:", asm, re.M).end():].split(".Lfunc_end", 1)[0].splitlines()
    for i, line in enumerate(lines):
        if not line.strip().startswith("s_barrier"):
            continue
        block = []
        for before in reversed(lines[:i]):
            before = before.strip()
            if re.match(r"\.LBB|s_c?branch|s_barrier", before):
                break
            block.append(before)
        yield block


def waits(block):
    """No LDS operation of the wave is in flight at the barrier, or the next step's bound, read behind the stores of the step before, has arrived:
    the register that it is handed over in is written in front of the barrier."""
    for i, line in enumerate(block):
        taken = re.match(r"; bound of the next step: (s\d+)$", line)
        if taken:
            return any(x.startswith(f"v_readfirstlane_b32 {taken[1]},") for x in block[i:])
        if line.startswith("ds_"):
            return False
        if re.match(r"s_waitcnt\b.*lgkmcnt\(0\)", line):
            return True
    return False


def test_a_wave_waits_before_every_barrier(tmp_path):
    out = str(tmp_path / "band_sweep.s")
    src = os.path.join(lib_build.CSRC, "band_sweep.hip")
    subprocess.check_call(["hipcc", *lib_build.FLAGS, "-S", "--cuda-device-only", src, "-o", out], stderr=subprocess.DEVNULL)
    asm = open(out).read()
    for form in ("k_band_sweepILb0E", "k_band_sweepILb1E"):
        found = list(barriers(asm, form))
        assert len(found) > 10, form
        for i, block in enumerate(found):
            assert waits(block), (form, i, block[:12])
