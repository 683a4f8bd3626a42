"""Inline assembly in the kernels: a scalar register that a vector instruction writes (a comparison's result, a
carry) is read by another vector instruction three instructions later at the earliest.  The hardware needs
two wait states in between, and the compiler, which adds them to its own code, adds none inside a block."""
import pathlib
import re

import pytest

CSRC = pathlib.Path(__file__).resolve().parent.parent / "paper_2204_03643_amd" / "csrc"


def asm_blocks():
    for path in sorted(CSRC.iterdir()):
        text = path.read_text()
        for m in re.finditer(r'\basm(?:\s+volatile)?\s*\(((?:\s*"(?:[^"\\]|\\.)*")+)', text):
            code = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', m.group(1)))
            lines = [l.strip() for l in code.replace("\\n", "\n").replace("\\t", " ").split("\n") if l.strip()]
            if lines:
                yield "%s:%d" % (path.name, text.count("\n", 0, m.start()) + 1), lines


def scalar_reads_and_writes(line):
    """Scalar operands that a comparison or an addition with carry reads, and the one it writes."""
    op, _, rest = line.partition(" ")
    args = [a.strip() for a in rest.split(",")]
    if op.startswith("v_cmp"):
        return [], args[0]
    if re.match(r"v_(add|sub|subrev)c_co_", op):
        return [args[4]], args[1]
    if re.match(r"v_(add|sub|subrev)_co_", op):
        return [], args[1]
    if op.startswith("v_cndmask"):
        return [args[3]], None
    if op == "s_nop":
        return [], None
    raise AssertionError("an instruction this test does not know: " + line)


def too_early(lines):
    """Pairs of instructions with fewer than two wait states between a scalar's write and its read."""
    written, at, found = {}, 0, []
    for line in lines:
        reads, write = scalar_reads_and_writes(line)
        found += [(lines[written[r][1]], line) for r in reads if r in written and at - written[r][0] < 3]
        if write:
            written[write] = (at, lines.index(line))
        at += 1 + (int(line.split()[1]) if line.startswith("s_nop") else 0)
    return found


def test_the_rule_itself():
    assert too_early(["v_cmp_gt_f32 vcc, %1, %2", "v_addc_co_u32 %0, vcc, %0, %0, vcc"])
    assert not too_early(["v_cmp_gt_f32 vcc, %1, %2", "s_nop 1", "v_addc_co_u32 %0, vcc, %0, %0, vcc"])


@pytest.mark.parametrize("where,lines", [pytest.param(w, l, id=w) for w, l in asm_blocks()])
def test_carries_are_not_read_too_early(where, lines):
    assert too_early(lines) == []
