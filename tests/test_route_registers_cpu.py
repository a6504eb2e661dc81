"""Registers of the router kernels, from the metadata that the compiler writes: what the launch rules count on."""
import os
import re
import subprocess

import pytest

from paper_2604_23108_amd import build


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """mangled name -> (vector registers, spilled vector registers) of every kernel of route.hip"""
    out = tmp_path_factory.mktemp("route") / "route.s"
    subprocess.run(["hipcc", *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "route.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    found = {}
    for entry in re.split(r"\n  - \.agpr_count:", out.read_text())[1:]:
        name = re.search(r"\.name:\s+(\S+)", entry).group(1)
        found[name] = (int(re.search(r"\.vgpr_count:\s+(\d+)", entry).group(1)),
                       int(re.search(r"\.vgpr_spill_count:\s+(\d+)", entry).group(1)))
    return found


def _of(kernels, pattern):
    hit = [v for k, v in kernels.items() if re.search(pattern, k)]
    assert hit, pattern
    return hit


def test_fp32_two_token_tiles_leave_room_for_a_second_workgroup(kernels):
    """Eight waves per workgroup, two workgroups per compute unit: four waves per SIMD, 128 registers each."""
    (regs, spilled), = _of(kernels, r"route_kernelILb0ELi2ELi1E")
    assert regs <= 128 and spilled == 0


def test_nothing_spills(kernels):
    """route_kernel takes two token tiles with at most two tiles of router rows: wider ones would not fit, and are not built."""
    assert len(_of(kernels, r"route_kernelILb")) == 2 * (4 + 2)
    for name, (_, spilled) in kernels.items():
        assert spilled == 0, name


def test_prefill_kernels_that_select_leave_room_for_a_second_workgroup(kernels):
    selecting = _of(kernels, r"route_prefill_kernelILi[24]ELi[123]ELb1E")
    assert len(selecting) == 5
    for regs, spilled in selecting:
        assert regs <= 128 and spilled == 0
