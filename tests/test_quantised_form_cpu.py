"""Which kernel the quantised decode calls take: a shape on either side of every line of the rule (host code only)."""
import pytest

import paper_2604_23108_amd as M
from paper_2604_23108_amd import bench_binding as BB

STAGED, SPLIT, DIRECT = 0, 1, 2
LARGE = dict(d=4096, n_groups=4, experts_per_group=16, d_ff=(768, 1024, 1536, 2048), k_groups=2, k_experts=4)
MID = dict(d=2048, n_groups=3, experts_per_group=8, d_ff=(512, 1024, 1536), k_groups=2, k_experts=4)
MANY = dict(d=2048, n_groups=4, experts_per_group=32, d_ff=(384, 384, 512, 384), k_groups=2, k_experts=4)
ODD = dict(d=1344, n_groups=5, experts_per_group=5, d_ff=(192, 448, 704, 960, 1216), k_groups=2, k_experts=4)
WIDE = dict(d=2560, n_groups=2, experts_per_group=32, d_ff=(1088, 1728), k_groups=2, k_experts=6)
FEW = dict(d=4096, n_groups=1, experts_per_group=2, d_ff=(8192,), k_groups=1, k_experts=1)
NARROW = dict(d=2048, n_groups=2, experts_per_group=32, d_ff=(256, 320), k_groups=2, k_experts=4)


@pytest.mark.parametrize("bits,shape,T,form", [
    (8, LARGE, 1, DIRECT), (8, LARGE, 2, SPLIT), (8, LARGE, 30, SPLIT), (8, LARGE, 31, STAGED),
    (8, MID, 3, DIRECT), (8, MID, 7, SPLIT), (8, MID, 24, SPLIT), (8, MID, 32, STAGED),
    (8, MANY, 3, DIRECT), (8, MANY, 25, SPLIT), (8, MANY, 26, STAGED),
    (8, ODD, 32, DIRECT), (8, WIDE, 20, SPLIT), (8, WIDE, 21, STAGED), (8, FEW, 32, DIRECT), (8, NARROW, 12, DIRECT),
    (4, LARGE, 5, SPLIT), (4, LARGE, 8, STAGED), (4, MID, 7, SPLIT), (4, MID, 9, STAGED),
    (4, ODD, 32, SPLIT), (4, WIDE, 20, SPLIT), (4, WIDE, 21, STAGED), (4, FEW, 3, SPLIT), (4, FEW, 7, STAGED),
])
def test_form_by_size(bits, shape, T, form):
    cfg = M.Config(T=T, select_mode=M.SELECT_GLOBAL, dtype=M.BF16, **shape)
    assert BB.mohge_bench_quantised_form(cfg, bits) == form


def test_refusals():
    base = dict(MID, select_mode=M.SELECT_GLOBAL)
    for kw, bits in ((dict(T=33, dtype=M.BF16), 8), (dict(T=0, dtype=M.BF16), 8), (dict(T=4, dtype=M.F32), 8), (dict(T=4, dtype=M.BF16), 16)):
        with pytest.raises(M.MohgeError):
            BB.mohge_bench_quantised_form(M.Config(**base, **kw), bits)
