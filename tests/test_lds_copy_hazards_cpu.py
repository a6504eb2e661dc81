"""Copies to LDS are inline assembly, which the compiler's hazard recognizer does not look into: what it put in front of them."""
import os
import re
import subprocess

import pytest

from paper_2604_23108_amd import build
from paper_2604_23108_amd.lds_hazards import hazards, hazards_of_file


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
    copies, bad = hazards_of_file(out)
    assert copies > 1000
    assert not bad, bad[:5]


def test_every_source_with_such_copies_is_looked_through():
    of = [f for f in os.listdir(build.CSRC) if re.search(r'"[^"\n]*global_load_lds[^"\n]*"', open(os.path.join(build.CSRC, f)).read())]
    assert sorted(of) == sorted(build.LDS_COPY_SOURCES)


PLANTED = """#include <hip/hip_runtime.h>
#ifndef MOHGE_LDS_COPY_NOP
#define MOHGE_LDS_COPY_NOP "0"
#endif
__global__ void k(const void* p, int i) {
  asm volatile("v_readfirstlane_b32 s4, %0\\n\\ts_mov_b32 s5, 0\\n\\ts_nop " NOP "\\n\\tglobal_load_lds_dwordx4 %0, s[4:5]"
               ::"v"(i), "{m0}"(0) : "memory", "s4", "s5");
}
"""


@pytest.mark.parametrize("nop,ends_well", [("MOHGE_LDS_COPY_NOP", True), ('"0"', False)])
def test_build_answers_a_copy_too_early_with_more_wait_states(tmp_path, monkeypatch, nop, ends_well):
    """A planted one is compiled again with the wait states it needs; where that does not help the build fails."""
    (tmp_path / "planted.hip").write_text(PLANTED.replace("NOP \"\\n", nop + " \"\\n", 1))
    for name in ("CSRC", "OBJDIR"):
        monkeypatch.setattr(build, name, str(tmp_path))
    monkeypatch.setattr(build, "LDS_COPY_SOURCES", ["planted.hip"])
    if ends_well:
        copies, bad = hazards_of_file(build.device_assembly(build._compile("planted.hip")))
        assert copies == 1 and not bad
    else:
        with pytest.raises(RuntimeError, match="too early"):
            build._compile("planted.hip")
