"""Inline assembly of the HIP sources: where a block of several instructions
has inputs beside its outputs, an output is written before the last input is
read, so it must be early-clobber ("&"), or the compiler may give an input of
the same value the output's register."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_08491_amd", "csrc")


def _blocks(text):
    """(line, body) of every asm statement, by its closing parenthesis."""
    text = re.sub(r"//[^\n]*", "", text)
    for m in re.finditer(r"\basm\s*(?:volatile\s*)?\(", text):
        depth, i, quoted = 1, m.end(), False
        while depth:
            c = text[i]
            if c == '"' and text[i - 1] != "\\":
                quoted = not quoted
            elif not quoted:
                depth += (c == "(") - (c == ")")
            i += 1
        yield text.count("\n", 0, m.start()) + 1, text[m.end():i - 1]


def _sections(body):
    """template, outputs, inputs: split at the colons outside of strings."""
    parts, quoted, last = [], False, 0
    for i, c in enumerate(body):
        if c == '"' and body[i - 1] != "\\":
            quoted = not quoted
        elif c == ":" and not quoted:
            parts.append(body[last:i])
            last = i + 1
    return (parts + [body[last:]] + ["", ""])[:3]


@pytest.mark.parametrize("name", sorted(n for n in os.listdir(CSRC) if n.endswith((".hip", ".h"))))
def test_outputs_written_before_the_last_input_is_read(name):
    for line, body in _blocks(open(os.path.join(CSRC, name)).read()):
        template, outputs, inputs = _sections(body)
        several = "SNP_" in template or template.count("\\n") > 1
        if several and inputs.strip():
            constraints = re.findall(r'"([^"]*)"\s*\(', outputs)
            assert constraints and all("&" in c for c in constraints), f"{name}:{line}: {constraints}"
