"""Inline assembly in the kernel sources: what it does to registers the compiler also uses has to be in its constraints."""
import glob
import os
import re

import paper_2604_23108_amd as M

CSRC = os.path.join(os.path.dirname(M.lib_path()), "csrc")


def _statements():
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.h"))):
        text = re.sub(r"//[^\n]*", "", open(path).read())
        for m in re.finditer(r"\basm\b\s*(volatile)?\s*\(", text):
            depth, i = 1, m.end()
            while depth:
                depth += {"(": 1, ")": -1}.get(text[i], 0)
                i += 1
            yield os.path.basename(path), text[m.start():i]


def test_m0_is_an_operand_where_assembly_uses_it():
    """A copy to LDS takes its destination from M0.  The compiler uses M0 for its own copies to LDS: a statement that
    sets it behind the compiler's back would send one of them elsewhere."""
    found = 0
    for path, stmt in _statements():
        code = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', stmt.split("::")[0]))
        if re.search(r"load_lds|\blds\b", code):
            found += 1
            assert '"{m0}"(' in stmt, f"{path}: copy to LDS without M0 as an operand: {stmt}"
        assert not re.search(r"\bm0\b", code), f"{path}: M0 written inside the statement: {stmt}"
    assert found >= 2
