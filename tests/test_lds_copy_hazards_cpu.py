"""Copies to LDS are inline assembly, which the compiler's hazard recognizer does not look into: what it put in front of them."""
import os
import re
import subprocess

from paper_2604_23108_amd import build

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


def test_the_look_back_finds_what_it_looks_for():
    near = ["v_readlane_b32 s4, v1, 3", "s_mov_b32 m0, s9", "s_nop 0", "global_load_lds_dwordx4 v2, s[4:5]"]
    assert len(hazards(near)[1]) == 1
    assert not hazards(["s_add_u32 s4, s4, s6", "s_mov_b32 m0, s9", "s_nop 0", "v_add_u32_e32 v2, s9, v2", "v_mov_b32_e32 v3, 0",
                        "v_mov_b32_e32 v4, 0", "global_load_lds_dwordx4 v2, s[4:5]"])[1]
    assert len(hazards(["v_nop"] * 5 + ["s_mov_b32 m0, s9", "global_load_lds_dwordx4 v[2:3], off"])[1]) == 1
    jump = ["v_readfirstlane_b32 s4, v1", "s_cbranch_scc1 .L1", "s_mov_b32 s4, 0", "s_nop 4", ".L1:", "s_nop 1", "global_load_lds_dwordx4 v2, s[4:5]"]
    assert len(hazards(jump)[1]) == 1


def test_no_copy_reads_a_scalar_register_too_early(tmp_path):
    out = tmp_path / "ffn_tiled.s"
    subprocess.run(["hipcc", *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "ffn_tiled.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    lines = [re.sub(r"[;/].*", "", l).strip() for l in out.read_text().split("\n")]
    copies, bad = hazards([l for l in lines if l and (l.endswith(":") or not l.startswith((".", "#")))])
    assert copies > 1000
    assert not bad, bad[:5]
