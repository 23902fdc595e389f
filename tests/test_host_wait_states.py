"""Row-broadcast FMAs of the distorted-mesh streaming (no GPU): the compiler
places no wait states for instructions inside inline assembly, so the code it
emits around them is read here.  Compiles csrc/stream_mapped.hip to assembly."""
import os
import re
import subprocess

import pytest

from paper_2012_05537_amd import build

WAIT_STATES = 2          # between a vector write of a register and a row broadcast FMA that reads it


def _regs(tok):
    m = re.match(r"v\[(\d+):(\d+)\]$", tok.strip())
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.match(r"v(\d+)$", tok.strip())
    return {int(m[1])} if m else set()


def violations(lines):
    """(number of row-broadcast FMAs, [(kernel, instruction, operand written too shortly before)])."""
    kernel, hist, count, bad = "", [], 0, []       # hist: (wait states, registers written)
    for line in lines:
        if re.match(r"_Z\w+:", line):
            kernel, hist = line.split(":")[0], []
        s = line.split(";")[0].strip()
        if not s or s.startswith(".") or s.endswith(":"):
            continue
        op, _, rest = s.partition(" ")
        ops = rest.replace(" row_newbcast", ", row_newbcast").split(",")
        if "row_newbcast" in s:
            count += 1
            states = 0
            for n, written in reversed(hist):
                if states >= WAIT_STATES:
                    break
                for name, tok in zip(("sum", "value", "weight"), ops):
                    if _regs(tok) & written:
                        bad.append((kernel, s, name))
                states += n
        n = int(rest, 0) + 1 if op == "s_nop" else 1
        hist = (hist + [(n, _regs(ops[0]) if op.startswith("v_") else set())])[-4:]
    return count, bad


def test_parser_sees_a_short_distance():
    fma = "v_fmac_f64_dpp v[0:1], v[2:3], v[4:5] row_newbcast:3 row_mask:0xf bank_mask:0xf"
    assert violations(["v_mov_b32_e32 v3, v9", "s_nop 0", fma])[1][0][2] == "value"
    assert violations(["v_mov_b32_e32 v3, v9", "s_nop 1", fma]) == (1, [])
    assert violations([fma, fma])[1][0][2] == "sum"


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="hipcc not available")
def test_row_broadcast_fmas_keep_their_distance(tmp_path):
    out = os.path.join(tmp_path, "stream_mapped.s")
    subprocess.check_call([build.HIPCC, *build.COMMON, "-S", "--offload-device-only",
                           os.path.join(build.CSRC, "stream_mapped.hip"), "-o", out], stderr=subprocess.DEVNULL)
    with open(out) as f:
        count, bad = violations(f)
    assert count >= 2 * 2 * sum((p + 1) ** 3 for p in range(3, 7))     # f and g, both storage types
    assert not bad, bad[:5]
