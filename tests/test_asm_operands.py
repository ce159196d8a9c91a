"""Assembly of several instructions writes its outputs before it has read all its inputs: outputs in vector registers are early clobbers, or the
compiler may give an input of the same value the register of an output."""
import glob
import os
import re

from paper_2306_03725_amd import build


def statements(text):
    for found in re.finditer(r"\basm volatile\s*\(", text):
        depth, at, quoted = 1, found.end(), False
        while depth:
            c = text[at]
            if c == '"' and text[at - 1] != "\\":
                quoted = not quoted
            elif not quoted:
                depth += (c == "(") - (c == ")")
            at += 1
        yield text[found.end():at - 1]


def test_outputs_of_several_instructions_are_early_clobbers():
    seen, late = 0, []
    for path in sorted(glob.glob(os.path.join(build.CSRC, "*.h*"))):
        with open(path) as fh:
            text = fh.read()
        for body in statements(text):
            if body.count("\\n") < 2:   # one instruction, or none
                continue
            seen += 1
            late += [(os.path.basename(path), o) for o in re.findall(r'"[+=]v"\([^)]*\)', body)]
    assert seen >= 3 and not late, late
