"""Inline assembly of the kernels: an output in a named register may share that register with an
input that is still to be read, unless it is written by the block's last instruction or marked
early-clobber."""
from __future__ import annotations

import pathlib
import re

CSRC = pathlib.Path(__file__).resolve().parent.parent / "paper_2510_03293_amd" / "csrc"


def asm_statements(text):
    """(template, outputs) of every asm statement: its instructions, and what follows the first
    colon outside the strings."""
    for m in re.finditer(r"\basm\s*(?:volatile)?\s*\(", text):
        depth, i, quoted, colons = 1, m.end(), False, []
        while depth:
            ch = text[i]
            if ch == '"' and text[i - 1] != "\\":
                quoted = not quoted
            elif not quoted:
                depth += {"(": 1, ")": -1}.get(ch, 0)
                if ch == ":":
                    colons.append(i)
            i += 1
        body = text[m.end():colons[0] if colons else i - 1]
        template = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', body))
        outputs = text[colons[0] + 1:colons[1] if len(colons) > 1 else i - 1] if colons else ""
        yield [x.strip() for x in re.split(r"\\n|;", template.replace("\\t", "")) if x.strip()], outputs


def hazards(text):
    bad = []
    for instructions, outputs in asm_statements(text):
        for constraint, reg in re.findall(r'"=([&]?)\{([^}]+)\}"', outputs):
            if not constraint and any(reg in x for x in instructions[:-1]):
                bad.append((reg, instructions))
    return bad


def test_the_check_sees_the_mistake():
    text = 'asm("v_cmp_ne_u32 s[92:93], 0, %[x]\\n\\t" "v_cmp_gt_u32 s[94:95], %[k], %[x]\\n\\t" : [o] "={s[92:93]}"(o) : [k] "s"(k));'
    assert hazards(text)
    assert not hazards(text.replace('"={s', '"=&{s'))


def test_outputs_in_named_registers_do_not_share_them_with_inputs():
    for path in sorted(CSRC.iterdir()):
        if path.suffix in (".h", ".hip"):
            assert not hazards(path.read_text()), path.name
