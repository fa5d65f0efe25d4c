"""Wait states in the generated code.  On gfx950 a scalar register that a vector instruction writes (v_cmp, v_readlane) may be
read as data by a vector instruction two wait states later, by a memory instruction as its address five, and as a lane number
four.  The compiler keeps this for its own instructions, not for those of inline assembly: so the sources whose assembly
holds such instructions are compiled here (no GPU needed) and looked over, line by line."""
import os
import re
import subprocess

import pytest

from paper_2508_02124_amd import build

SCALAR = re.compile(r"(?<![\w.])(?:(vcc(?:_lo|_hi)?)|s(\d+)|s\[(\d+):(\d+)\])(?![\w\[])")
TWO_RESULTS = re.compile(r"v_(add|sub|subrev|addc|subb|subbrev)_co_|v_div_scale|v_mad_[ui]64_")


def scalars(operands):
    found = set()
    for vcc, one, first, last in SCALAR.findall(",".join(operands)):
        if vcc:
            found |= {"vcc_lo", "vcc_hi"} if vcc == "vcc" else {vcc}
        else:
            found |= {f"s{i}" for i in range(int(first or one), int(last or one) + 1)}
    return found


def early_reads(lines):
    """(scalar registers written by vector instructions, reads of one that come too early), in the order of the text."""
    now, written, writes, early = 0, {}, 0, []
    for number, line in enumerate(lines, 1):
        text = line.split(";")[0].strip()
        if re.match(r"[\w$]+:", text):  # another function
            written = {}
        m = re.match(r"((?:v|s|ds|global|buffer|flat|scratch)_\w+)\s*(.*)", text)
        if not m:
            continue
        op, operands = m[1], re.split(r",(?![^\[]*\])", m[2])
        if op == "s_nop":
            now += int(operands[0], 0) + 1
            continue
        now += 1
        vector, memory = op.startswith("v_"), not op.startswith(("v_", "s_", "ds_"))
        results = 0 if memory else 2 if TWO_RESULTS.match(op) else 1
        for reg in scalars(operands[results:]) & written.keys():
            lane = op.startswith(("v_readlane", "v_writelane")) and reg in scalars(operands[2:])
            wait = now - written[reg] - 1
            if wait < (5 if memory else 4 if lane else 2 if vector else 0):
                early.append(f"line {number}: {text} ({reg} written {wait} wait states before)")
        for reg in scalars(operands[:results]):
            if vector:
                written[reg] = now
                writes += 1
            else:
                written.pop(reg, None)
    return writes, early


def test_what_counts_as_early():
    write = "v_cmp_le_i32_e32 vcc, v5, v18"
    to_lane, load = "v_writelane_b32 v0, vcc_lo, 1", "global_load_dwordx4 v[0:3], v4, vcc"
    for between, read, ok in (([], to_lane, False), (["v_add_u32 v1, 1, v1"], to_lane, False), (["s_nop 1"], to_lane, True),
                              (["s_nop 1"], "v_writelane_b32 v0, s3, vcc_lo", False), (["s_nop 3"], load, False),
                              (["s_nop 4"], load, True), (["s_mov_b64 vcc, 0"], to_lane, True),
                              ([], "s_mov_b32 s3, vcc_lo", True)):
        writes, early = early_reads([write, *between, read])
        assert writes == 2 and bool(early) != ok, (between, read, early)


@pytest.mark.parametrize("source", ["select.hip", "fwd.hip", "bwd.hip"])
def test_scalars_are_read_late_enough(source):
    r = subprocess.run([build._hipcc(), *build.FLAGS, *build.EXTRA_FLAGS.get(source, []), "--cuda-device-only", "-S",
                        os.path.join(build.CSRC, source), "-o", "-"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    writes, early = early_reads(r.stdout.splitlines())
    assert writes > 1000
    assert not early, f"{len(early)} of {writes}: " + "; ".join(early[:3])
