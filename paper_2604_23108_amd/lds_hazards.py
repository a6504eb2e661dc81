"""Copies to LDS are inline assembly in some kernels, which the compiler's hazard recognizer does not look into.  This looks through
the assembly that it made for what it put in front of them."""
from __future__ import annotations

import re

WAIT_STATES = 5          # between a vector instruction that writes a scalar register and a memory access that reads it


def _scalars(text):
    found = {"m0"} if re.search(r"\bm0\b", text) else set()
    for lo, hi, one in re.findall(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b", text):
        found |= {f"s{one}"} if one else {f"s{i}" for i in range(int(lo), int(hi) + 1)}
    return found


def hazards(lines):
    """The number of copies, and those whose M0 or base a vector instruction wrote less than WAIT_STATES before on some path,
    or whose M0 the instruction right before them wrote."""
    jumps = {}
    for i, line in enumerate(lines):
        if line.startswith(("s_cbranch", "s_branch")):
            jumps.setdefault(line.split()[1], []).append(i)

    def before(i):
        """Indices of the instructions that may run right before line i."""
        todo, seen, found = [i - 1], set(), []
        while todo:
            k = todo.pop()
            if k < 0 or k in seen:
                continue
            seen.add(k)
            if lines[k].endswith(":"):
                todo += [k - 1]
                found += jumps.get(lines[k][:-1], [])
            elif not (lines[k].startswith(("s_branch", "s_endpgm", "s_setpc")) and k + 1 < len(lines) and lines[k + 1].endswith(":")):
                found.append(k)
        return found

    bad, copies = [], 0
    for i, line in enumerate(lines):
        if not line.startswith("global_load_lds"):
            continue
        copies += 1
        reads = _scalars(line.split(None, 1)[1]) | {"m0"}
        todo, seen = [(k, 0) for k in before(i)], set()
        while todo:
            k, states = todo.pop()
            if (k, states) in seen or states >= WAIT_STATES:
                continue
            seen.add((k, states))
            op, _, rest = lines[k].replace("\t", " ").partition(" ")
            if op == "s_nop":
                todo += [(q, states + int(rest, 0) + 1) for q in before(k)]
                continue
            written = _scalars(rest.split(",")[0])
            if written & reads and (op.startswith("v_") or (states == 0 and "m0" in written)):
                bad.append((lines[k], line))
            todo += [(q, states + 1) for q in before(k)]
    return copies, bad


def hazards_of_file(path):
    """hazards() of the assembly in a file."""
    with open(path) as f:
        lines = [re.sub(r"[;/].*", "", l).strip() for l in f.read().split("\n")]
    return hazards([l for l in lines if l and (l.endswith(":") or not l.startswith((".", "#")))])
