"""Registers of the bf16 tile kernels, from the assembly and the metadata that the compiler writes."""
import os
import re
import subprocess

import pytest

from paper_2604_23108_amd import build


@pytest.fixture(scope="module")
def text(tmp_path_factory):
    built = build.device_assembly(os.path.join(build.OBJDIR, "ffn_tiled.o"))
    newest = max(os.path.getmtime(os.path.join(build.CSRC, f)) for f in os.listdir(build.CSRC))
    if not os.path.exists(built) or os.path.getmtime(built) < newest:
        built = str(tmp_path_factory.mktemp("tiled") / "ffn_tiled.s")
        subprocess.run(["hipcc", *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "ffn_tiled.hip"), "-o", built],
                       check=True, capture_output=True)
    with open(built) as f:
        return f.read()


@pytest.fixture(scope="module")
def kernels(text):
    """mangled name -> spilled vector registers"""
    return {re.search(r"\.name:\s+(\S+)", e).group(1): int(re.search(r"\.vgpr_spill_count:\s+(\d+)", e).group(1))
            for e in re.split(r"\n  - \.agpr_count:", text)[1:]}


def test_few_registers_spill(kernels):
    """The big form has every register in use: what little it spills is constant over a tile.  The small form has room."""
    big = {n: s for n, s in kernels.items() if re.search(r"ffn_(fused|tile)_kernel", n)}
    small = {n: s for n, s in kernels.items() if "ffn_small" in n}
    assert len(big) == 4 + 6 + 3 and len(small) == 6 + 2 + 2
    assert all(s <= 16 for s in big.values()), big
    assert all(s == 0 for s in small.values()), small


def loops_with_products(lines):
    """Line ranges of the innermost loops that hold MFMAs."""
    at = {l[:-1]: i for i, l in enumerate(lines) if l.endswith(":")}
    found = []
    for i, l in enumerate(lines):
        m = re.match(r"s_c?branch\w*\s+(\S+)", l)
        if m and at.get(m.group(1), i) < i and any(x.startswith("v_mfma") for x in lines[at[m.group(1)]:i]):
            found.append((at[m.group(1)], i))
    return [(a, b) for a, b in found if not any((c, d) != (a, b) and a <= c and d <= b for c, d in found)]


def test_main_loops_keep_out_of_private_memory(text):
    """None of them reads any, and only the second projection by itself (mohge_expert_ffn_down), whose full tiles keep four
    registers there, writes once per stage of 64 MFMAs."""
    checked = 0
    for body in re.findall(r"^_ZN\S*ffn_(?:fused|tile|small)\S*:.*?^\.Lfunc_end", text, re.M | re.S):
        lines = [re.sub(r"[;/].*", "", l).strip() for l in body.split("\n")]
        lines = [l for l in lines if l and (l.endswith(":") or not l.startswith("."))]
        for a, b in loops_with_products(lines):
            loop = lines[a:b]
            checked += 1
            private = [l for l in loop if l.startswith("scratch_")]
            assert len([l for l in loop if l.startswith("v_mfma")]) >= 16
            if re.search(r"ffn_tile_kernelILi1E", lines[0]):
                assert len(private) <= 1 and all(l.startswith("scratch_store") for l in private), (lines[0], a, b)
            else:
                assert not private, (lines[0], a, b)
    assert checked >= 50
