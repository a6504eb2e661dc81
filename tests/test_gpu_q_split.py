"""Decode with quantised weights in every kernel form (staged, split and, for FP8, direct): rows per expert around the
passes and chunks of the staged tokens, reductions that leave waves without indices or end in half a unit, column blocks
cut short; against float64 on the dequantised weights.  The form is an argument here, whatever the rule by size."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

EDGES = [(counts, d, ff) for counts in [(0, 1, 0, 0), (1, 0, 15, 16), (17, 2, 0, 9), (4, 3, 5, 8), (0, 32, 0, 0)]
         for d, ff in [(64, (64, 128)), (192, (320, 64)), (1088, (192, 448)), (2112, (1088, 576)), (4096, (64, 832))]]
FORMS = {"staged": 0, "split": 1, "direct": 2}


def _value(kind, codes, scale):
    if kind == "fp8":
        return codes.view(torch.float8_e4m3fn).cpu().double() * scale.cpu().double().unsqueeze(-1)
    table = torch.tensor([0, .5, 1, 1.5, 2, 3, 4, 6, -0.0, -.5, -1, -1.5, -2, -3, -4, -6], dtype=torch.float64)
    c = codes.cpu().long()
    v = torch.stack([table[c & 15], table[c >> 4]], -1).flatten(-2)
    s = torch.pow(2.0, scale.cpu().double() - 127).repeat_interleave(32, -1)
    return v * s


def _check(kind, form, T, d, n, d_ff, eidx):
    import paper_2604_23108_amd as M
    from paper_2604_23108_amd import bench_binding as BB
    Ne, k = 2 * n, eidx.shape[1]
    gen = torch.Generator(device="cuda").manual_seed(T + d)
    normal = lambda *s: torch.randn(s, generator=gen, device="cuda")
    cfg = M.Config(T=T, d=d, n_groups=2, experts_per_group=n, d_ff=d_ff, k_groups=k, k_experts=k,
                   select_mode=M.SELECT_PER_GROUP, dtype=M.BF16)
    x = normal(T, d).bfloat16()
    w13 = [(normal(n, 2 * f, d) * 0.05).bfloat16() for f in d_ff]
    w2 = [(normal(n, d, f) * 0.05).bfloat16() for f in d_ff]
    L = M.MoHGELayer(cfg, normal(2, d) * 0.02, normal(Ne, d) * 0.02, w13, w2)
    L.use_fp8_weights() if kind == "fp8" else L.use_mxfp4_weights()
    q, bits = (L.w8, 8) if kind == "fp8" else (L.w4, 4)
    M.mohge_permute(cfg, torch.from_numpy(eidx).cuda(), L.counts, L.offsets, L.perm, L.inv_perm, None, None, L.ws_permute)
    L.y_perm.fill_(float("nan"))
    BB.mohge_bench_expert_ffn_quantised(cfg, x, L.perm, L.offsets, *q, L.y_perm, L.ws_ffn, bits, FORMS[form])
    torch.cuda.synchronize()
    off, tok, xs = L.offsets.tolist(), L.perm.cpu().long() // k, x.cpu().double()
    want = torch.zeros((T * k, d), dtype=torch.float64)
    for e in range(Ne):
        lo, hi = off[e], off[e + 1]
        if hi > lo:
            g, i = divmod(e, n)
            a, b = (xs[tok[lo:hi]] @ _value(kind, q[0][g][i], q[1][g][i]).T).split(d_ff[g], dim=1)
            want[lo:hi] = (a * torch.sigmoid(a) * b) @ _value(kind, q[2][g][i], q[3][g][i]).T
    got = L.y_perm.cpu().double()
    assert torch.isfinite(got).all()
    # the dequantised weights are exact in bf16; h and y are rounded to bf16 once each: 2^-9 of the value and of a sum of
    # such terms
    assert (got - want).abs().max() <= 8e-3 * want.abs().max()


@pytest.mark.parametrize("kind,form", [("fp8", "staged"), ("fp8", "split"), ("fp8", "direct"), ("mxfp4", "staged"), ("mxfp4", "split")])
@pytest.mark.parametrize("counts,d,d_ff", EDGES)
def test_kernel_edges(kind, form, counts, d, d_ff):
    eidx = np.random.default_rng(5).permutation(np.repeat(np.arange(4), counts)).astype(np.int32).reshape(-1, 1)
    print(f"[quantised] {kind} {form} counts={counts} d={d} d_ff={d_ff}", flush=True)
    _check(kind, form, sum(counts), d, 2, d_ff, eidx)
