"""Inline assembly of several instructions in the kernels' sources: every output
is written before later instructions read their inputs, so each has to be marked
early-clobber ("=&", "+&"); without the mark the compiler may hold an input of
the same value in the output's register."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1702_05156_amd", "csrc")
FILES = sorted(glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(CSRC, "*.hip")))


def _blocks(text):
    """(line, template, [output constraints]) of each asm statement."""
    for m in re.finditer(r"\basm\s*(?:volatile\s*)?\(", text):
        depth, i, quoted = 1, m.end(), False
        while depth:
            c = text[i]
            if quoted:
                i += c == "\\"
                quoted = c != '"'
            else:
                quoted = c == '"'
                depth += (c == "(") - (c == ")")
            i += 1
        body = text[m.end():i - 1]
        parts = re.split(r":(?=(?:[^\"]*\"[^\"]*\")*[^\"]*$)", body)
        template = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', parts[0]))
        outputs = re.findall(r'"([^"]*)"\s*\(', parts[1]) if len(parts) > 1 else []
        yield text.count("\n", 0, m.start()) + 1, template, outputs


def test_the_scan_sees_blocks():
    text = 'asm("v_mov_b32 %0, %1\\n\\t" "v_add %0, %0, %2" : "+v"(a) : "v"(b), "v"(f(c)));'
    assert list(_blocks(text)) == [(1, "v_mov_b32 %0, %1\\n\\tv_add %0, %0, %2", ["+v"])]
    assert sum(len(list(_blocks(open(f).read()))) for f in FILES) > 10


@pytest.mark.parametrize("path", FILES, ids=os.path.basename)
def test_outputs_of_several_instructions_are_early_clobber(path):
    bad = []
    for line, template, outputs in _blocks(open(path).read()):
        code = [s for s in re.split(r"\\n\\t|\\n", template) if s.strip() and not s.strip().startswith(".")]
        if len(code) > 1:
            bad += [f"{os.path.basename(path)}:{line} {o}" for o in outputs if "&" not in o]
    assert not bad, bad
