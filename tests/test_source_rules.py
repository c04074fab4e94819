"""Rules that the device sources keep because no run shows reliably that one is broken."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_30033_amd", "csrc")


def asm_statements(text):
    """Every asm statement: (line, source of its parenthesis)."""
    text = re.sub(r"//[^\n]*", "", text)
    for m in re.finditer(r"\basm\s+(?:volatile\s*)?\(", text):
        depth, at = 1, m.end()
        while depth:
            depth += {"(": 1, ")": -1}.get(text[at], 0)
            at += 1
        yield text.count("\n", 0, m.start()) + 1, text[m.end():at - 1]


@pytest.mark.parametrize("name", sorted(n for n in os.listdir(CSRC) if n.endswith((".hip", ".h"))))
def test_loads_in_inline_assembly_wait_in_the_same_statement(name):
    # an output register counts as written when the statement ends: a load that is waited for elsewhere may be copied,
    # spilled or its register handed on before its data has arrived
    for line, body in asm_statements(open(os.path.join(CSRC, name)).read()):
        loads = list(re.finditer(r"\b(ds_read|ds_load|buffer_load|global_load|flat_load|scratch_load|s_load)\w*", body))
        if not loads:
            continue
        wait = "lgkmcnt(0)" if loads[-1].group(1) in ("ds_read", "ds_load", "s_load") else "vmcnt(0)"
        assert wait in body[loads[-1].end():], f"{name}:{line}"
        assert all("&" in c for c in re.findall(r'"(=[^"]*)"', body)), f"{name}:{line}: outputs early-clobber"
