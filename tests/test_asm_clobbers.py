"""Inline assembly must name every register it writes: the compiler may keep a value of its own in m0, scc, vcc or exec."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2503_01483_amd", "csrc")
# instructions whose first operand is not a destination
NO_DEST = re.compile(r"s_(nop|waitcnt|barrier|cmp|bitcmp|setprio|sleep|branch|cbranch)|buffer_load_\w+ .* lds|\w*store")


def _asm_statements():
    for name in sorted(os.listdir(CSRC)):
        text = open(os.path.join(CSRC, name)).read()
        for m in re.finditer(r"\basm\s*(?:volatile)?\s*\(", text):
            depth, i = 1, m.end()
            while depth:
                depth += {"(": 1, ")": -1}.get(text[i], 0)
                i += 1
            yield name, text[: m.start()].count("\n") + 1, text[m.end():i - 1]


def _written(code):
    for line in re.split(r"\\n(?:\\t)?", code):
        line = line.strip()
        if not line or NO_DEST.match(line):
            if line.startswith(("s_cmp", "s_bitcmp")):
                yield "scc"
            continue
        op, _, rest = line.partition(" ")
        dest = rest.split(",")[0].strip()
        if dest in ("m0", "vcc", "exec", "scc"):
            yield dest
        if re.match(r"s_(add|sub|and|or|xor|lsh|min|max)", op):
            yield "scc"


def test_every_special_register_written_is_a_clobber():
    seen = 0
    for name, line, body in _asm_statements():
        code = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', body.split(":")[0]))
        clobbers = re.findall(r'"(\w+)"', body.rsplit(":", 1)[1]) if body.count(":") >= 3 else []
        for reg in _written(code):
            seen += 1
            assert reg in clobbers, f"{name}:{line} writes {reg} and does not say so"
    assert seen >= 2     # the loads into LDS write m0 and scc


@pytest.mark.parametrize("code,regs", [("s_add_u32 m0, %1, %3\\n\\ts_nop 0\\n\\tbuffer_load_dwordx4 %0, %2, 0 offen lds", {"m0", "scc"}),
                                       ("s_nop 15", set()), ("s_mov_b32 m0, %0", {"m0"}), ("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0", set())])
def test_what_a_statement_writes(code, regs):
    assert set(_written(code)) == regs
