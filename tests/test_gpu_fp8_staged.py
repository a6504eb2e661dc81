"""FP8 decode through the kernel that stages an expert's tokens in LDS once per workgroup, taken here whatever the rule by size,
against float64 on the dequantised weights."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


# T, d, experts per group (two groups), widths, skewed: experts all with one or two rows; fewer rows than experts;
# up to 32 rows on one expert, a reduction of several staged chunks and widths that end in partial column blocks
@pytest.mark.parametrize("T,d,n,d_ff,skewed", [(32, 192, 16, (576, 704), False), (32, 1088, 8, (1216, 1344), False),
                                               (20, 192, 32, (1024, 1088), False), (32, 2112, 8, (1216, 1344), True),
                                               (25, 4096, 8, (1216, 1344), True)])
def test_fp8_staged_kernel(T, d, n, d_ff, skewed):
    import paper_2604_23108_amd as M
    from paper_2604_23108_amd import bench_binding as BB
    Ne, k = 2 * n, 2
    P = T * k
    gen = torch.Generator(device="cuda").manual_seed(T + d)
    normal = lambda *s: torch.randn(s, generator=gen, device="cuda")
    cfg = M.Config(T=T, d=d, n_groups=2, experts_per_group=n, d_ff=d_ff, k_groups=2, k_experts=k,
                   select_mode=M.SELECT_PER_GROUP, dtype=M.BF16)
    x = normal(T, d).bfloat16()
    w13 = [(normal(n, 2 * f, d) * 0.05).bfloat16() for f in d_ff]
    w2 = [(normal(n, d, f) * 0.05).bfloat16() for f in d_ff]
    L = M.MoHGELayer(cfg, normal(2, d) * 0.02, normal(Ne, d) * 0.02, w13, w2)
    L.use_fp8_weights()
    rng = np.random.default_rng(T)
    e0 = np.where(rng.random(T) < 0.8, 1, rng.integers(0, n, T)) if skewed else rng.integers(0, n, T)
    eidx = np.stack([e0, n + rng.integers(0, n, T)], 1).astype(np.int32)
    assert not skewed or (e0 == 1).sum() > 16                       # more rows than one block of 16
    print(f"[fp8 staged] T={T} d={d} skewed={skewed}", flush=True)
    M.mohge_permute(cfg, torch.from_numpy(eidx).cuda(), L.counts, L.offsets, L.perm, L.inv_perm, None, None, L.ws_permute)
    L.y_perm.fill_(float("nan"))
    BB.mohge_bench_expert_ffn_quantised(cfg, x, L.perm, L.offsets, *L.w8, L.y_perm, L.ws_ffn, 8, 0)
    torch.cuda.synchronize()
    c13, s13, c2, s2 = L.w8
    value = lambda c, s: c.view(torch.float8_e4m3fn).cpu().double() * s.cpu().double().unsqueeze(-1)
    off, tok, xs = L.offsets.tolist(), (L.perm.cpu().long() // k), x.cpu().double()
    want = torch.zeros((P, d), dtype=torch.float64)
    for e in range(Ne):
        lo, hi = off[e], off[e + 1]
        if hi > lo:
            g, i = divmod(e, n)
            a, b = (xs[tok[lo:hi]] @ value(c13[g][i], s13[g][i]).T).split(d_ff[g], dim=1)
            want[lo:hi] = (a * torch.sigmoid(a) * b) @ value(c2[g][i], s2[g][i]).T
    got = L.y_perm.cpu().double()
    assert torch.isfinite(got).all()
    # the codes are exact in bf16; h and y are rounded to bf16 once each: 2^-9 of the value and of a sum of such terms
    assert (got - want).abs().max() <= 8e-3 * want.abs().max()
