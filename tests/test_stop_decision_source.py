"""The stop decision inside a row launch must not store what that launch still
reads: workgroups, and wavefronts of one workgroup, may start after tile 0 has
recorded it, and a wavefront that left alone would leave the others with LDS
tables half filled.  Read off the sources, because the order of events that
shows the fault cannot be forced."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2103_10203_amd", "csrc")


def _body(text, start):
    """The braced block that follows the first match of `start`."""
    m = re.search(start, text)
    assert m, start
    i = text.index("{", m.end())
    depth, j = 0, i
    while True:
        depth += {"{": 1, "}": -1}.get(text[j], 0)
        j += 1
        if depth == 0:
            return text[i:j]


def _source(name):
    with open(os.path.join(CSRC, name)) as fh:
        return re.sub(r"//[^\n]*", "", fh.read())


def _stored_by_stop():
    return set(re.findall(r"\bS\.(\w+)\s*=[^=]", _body(_source("solve_kernels.h"), r"\bvoid stop_rve\(")))


def test_row_launches_read_nothing_the_decision_stores():
    stored = _stored_by_stop()
    assert {"status", "resid"} <= stored
    rule = set(re.findall(r"\bS\.(\w+)", _body(_source("solve_kernels.h"), r"\bint stop_rule\(")))
    rows = [_body(_source("solve_fast.h"), r"\bvoid row_tile\("), _body(_source("solve_cp.h"), r"\bk_row_cp\(")]
    for body in rows:
        read = set(re.findall(r"\bst\[b\]\.(\w+)", body))
        assert read and "stop_rve(" in body
        assert not stored & (read | rule), stored & (read | rule)


def test_column_and_axis1_launches_see_the_decision():
    stored = _stored_by_stop()
    for name, fn in (("solve_fast.h", r"\bvoid col_tile\("), ("solve_fast.h", r"\bk_mid_fast\("),
                     ("solve_kernels.h", r"\bk_col\("), ("solve_kernels.h", r"\bk_mid\(")):
        body = _body(_source(name), fn)
        first = re.search(r"if \([^\n]*\bst\[b\]\.(\w+)\)", body)
        assert first and first.group(1) in stored, fn
