"""What inline assembly in the kernels owes the compiler, which does not look inside it: SCC named
among the clobbers where an instruction writes it, and the two wait states that gfx950 wants between
a vector instruction that writes a carry (VCC or a scalar pair) and a vector instruction that takes
it in.  Read from the sources, without a GPU."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1404_3456_amd", "csrc")
SCC_WRITERS = re.compile(r"s_(and|or|xor|andn2|orn2|nand|nor|xnor|add|addc|sub|subb|lshl|lshr|ashr|not|"
                         r"bcnt\d|cmp|cmpk|bfe|min|max|abs|wqm)_")
WAIT_STATES = 2


def blocks():
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h*"))):
        text = re.sub(r"//[^\n]*", "", open(path).read())
        for m in re.finditer(r"\basm(?:\s+volatile)?\s*\((.*?)\)\s*;", text, re.S):
            body = m.group(1)
            code = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', body.split("\n        :")[0].split(": \"")[0]))
            lines = [x.strip() for x in code.replace("\\t", " ").split("\\n") if x.strip()]
            if lines:
                yield f"{os.path.basename(path)}:{text[:m.start()].count(chr(10)) + 1}", lines, body


def test_blocks_are_found():
    assert sum("v_subb_co_u32" in " ".join(lines) for _, lines, _ in blocks()) >= 2


@pytest.mark.parametrize("where, lines, body", list(blocks()), ids=lambda x: x if isinstance(x, str) and ".h" in x else "")
def test_block(where, lines, body):
    if any(SCC_WRITERS.match(x) for x in lines):
        assert re.search(r'"scc"\s*(,|$)', body.strip()), f"{where} writes SCC and does not say so"
    age = {}  # carry register -> wait states since a vector instruction wrote it
    for x in lines:
        op, _, rest = x.partition(" ")
        regs = [r.strip() for r in rest.split(",")]
        if op == "s_nop":
            states = int(regs[0]) + 1
        else:
            states = 1
            if re.match(r"v_(subb|addc|subbrev)_co_u32", op):
                assert age.get(regs[4], WAIT_STATES) >= WAIT_STATES, f"{where}: {x} takes in a fresh carry"
        age = {r: a + states for r, a in age.items()}
        if re.match(r"v_(sub|subb|add|addc|subrev|subbrev)_co_u32", op):
            age[regs[1]] = 0
        elif op.startswith("s_") and op != "s_nop":
            age.pop(regs[0], None)  # written by a scalar instruction: the hardware waits
