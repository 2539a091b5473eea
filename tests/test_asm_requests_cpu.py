"""The global->LDS requests that the kernels write as inline assembly: the compiler neither tracks
the M0 they write nor inserts wait states for them.  The statements have to name M0 as clobbered and
wait one state after writing it (a pass over the kernel sources), and in the code as compiled no
vector instruction may write a request's scalar base within five wait states before it."""
import glob
import os
import re
import subprocess

import pytest

from paper_2311_18677_amd import build

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2311_18677_amd", "csrc")


def statements():
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        text = open(path).read()
        for m in re.finditer(r"\basm\s+volatile\s*\((.*?)\);", text, re.S):
            if "global_load_lds" in m.group(1):
                yield pytest.param(m.group(1), id="%s:%d" % (os.path.basename(path), text.count("\n", 0, m.start()) + 1))


def test_there_are_some():
    assert len(list(statements())) >= 3


@pytest.mark.parametrize("asm", statements())
def test_m0_and_wait_states(asm):
    code, operands = asm.split("::", 1)
    lines = "".join(re.findall(r'"(.*?)"', code)).replace("\\t", "").split("\\n")
    load = next(i for i, x in enumerate(lines) if x.startswith("global_load_lds"))
    write = next(i for i, x in enumerate(lines) if x.startswith("s_mov_b32 m0"))
    assert load == len(lines) - 1 and write < load

    assert states(lines[write + 1:load]) >= 1
    clobbers = operands.rsplit(":", 1)[1]
    assert '"m0"' in clobbers and '"memory"' in clobbers


def states(instructions):
    return sum(int(x.split()[1]) + 1 if x.startswith("s_nop") else 1 for x in instructions)


def scalars(operand):
    """Numbers of the scalar registers that an operand names."""
    m = re.match(r"s\[(\d+):(\d+)\]$", operand) or re.match(r"s(\d+)$", operand)
    return set(range(int(m.group(1)), int(m.groups()[-1]) + 1)) if m else set()


def hazards(assembly):
    """(requests with a scalar base, those whose base a vector instruction wrote too late)"""
    seen, bad, found = [], [], 0
    for line in assembly.splitlines():
        text = line.split(";")[0].strip()
        if not text or text.startswith(".") or text.endswith(":"):
            continue
        ops = [x.strip() for x in text.split(None, 1)[1].split(",")] if " " in text or "\t" in text else []
        if text.startswith("global_load_lds"):
            base = scalars(ops[1].split()[0])
            if base:
                found += 1
                for k in range(len(seen) - 1, -1, -1):
                    if states([x for x, _ in seen[k + 1:]]) >= 5:
                        break
                    if seen[k][0].startswith("v_") and seen[k][1] and scalars(seen[k][1][0]) & base:
                        bad.append((seen[k][0], text))
        seen = (seen + [(text, ops)])[-8:]
    return found, bad


def test_the_pass_sees_a_late_write():
    late = "\tv_readfirstlane_b32 s5, v1\n\ts_mov_b32 m0, s9\n\ts_nop 0\n\tglobal_load_lds_dwordx4 v2, s[4:5]\n"
    assert hazards(late) == (1, [("v_readfirstlane_b32 s5, v1", "global_load_lds_dwordx4 v2, s[4:5]")])
    assert hazards(late.replace("s_nop 0", "s_nop 3"))[1] == []
    assert hazards(late.replace("s5, v1", "s6, v1"))[1] == []


@pytest.mark.parametrize("source", ["sw_prefill_mfma.hip", "sw_prefill_halves.hip", "sw_prefill_split.hip", "sw_decode_split.hip"])
def test_no_base_is_written_late(source):
    res = subprocess.run([build.HIPCC] + build.FLAGS + ["-S", "--cuda-device-only", "-o", "-", os.path.join(CSRC, source)],
                         capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr
    found, bad = hazards(res.stdout)
    assert found > 8 and not bad
