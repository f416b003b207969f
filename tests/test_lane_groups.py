"""The groups of lanes of the re-tessellation kernels exchange values by moves
between lanes (DPP), which read nothing of a lane that is switched off.  A call
of group_max, group_sum or group_or on the right of &&, || or ?: runs with only
the lanes that got there, so none may stand there (the result of a wrong one may
hide: a cell's mirrors left out too often are put back by a later check)."""
import os
import re

import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_1410_3219_amd", "csrc")


def conditional_moves(text):
    """(line, statement) of each such call behind a short circuit."""
    text = re.sub(r"//[^\n]*", "", text)
    out = []
    for m in re.finditer(r"\bgroup_(?:max|sum|or|min)(?:<\w+>)?\(", text):
        start = max(text.rfind(c, 0, m.start()) for c in ";{}") + 1
        before = text[start:m.start()]
        if re.search(r"&&|\|\||\?", before):
            out.append((text.count("\n", 0, m.start()) + 1, " ".join(before.split())))
    return out


@pytest.mark.parametrize("name", ["rich_retess.hip", "rich_kernels.hip"])
def test_no_lane_move_behind_a_short_circuit(name):
    assert conditional_moves(open(os.path.join(SRC, name)).read()) == []


def test_a_short_circuit_is_seen():
    assert conditional_moves("a = f();\n  b = l < 4 && x <= 4.0 * group_max(far2);")
    assert not conditional_moves("const double r = group_max(far2);\n  b = l < 4 && x <= r;")
