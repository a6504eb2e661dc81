"""Decode with quantised weights in both kernel forms (split reduction, staged), FP8 and MXFP4: rows per expert around the
passes and chunks of the staged tokens, reductions that leave waves without indices or end in half a unit, column blocks
cut short; against float64 on the dequantised weights."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

SPLIT = [(counts, d, ff) for counts in [(0, 1, 0, 0), (1, 0, 15, 16), (17, 2, 0, 9), (4, 3, 5, 8)]
         for d, ff in [(64, (64, 128)), (192, (320, 64)), (1088, (192, 448)), (4096, (64, 832))]]
# shapes that choose the staged kernel: experts of one or two rows, widths that end in partial column blocks
STAGED = [("fp8", 192, 64, (1600, 1728)), ("mxfp4", 1152, 64, (768, 896))]


def _value(kind, codes, scale):
    if kind == "fp8":
        return codes.view(torch.float8_e4m3fn).cpu().double() * scale.cpu().double().unsqueeze(-1)
    table = torch.tensor([0, .5, 1, 1.5, 2, 3, 4, 6, -0.0, -.5, -1, -1.5, -2, -3, -4, -6], dtype=torch.float64)
    c = codes.cpu().long()
    v = torch.stack([table[c & 15], table[c >> 4]], -1).flatten(-2)
    s = torch.pow(2.0, scale.cpu().double() - 127).repeat_interleave(32, -1)
    return v * s


def _check(kind, T, d, n, d_ff, eidx):
    import paper_2604_23108_amd as M
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
    q, call = (L.w8, M.mohge_expert_ffn_w8) if kind == "fp8" else (L.w4, M.mohge_expert_ffn_w4)
    M.mohge_permute(cfg, torch.from_numpy(eidx).cuda(), L.counts, L.offsets, L.perm, L.inv_perm, None, None, L.ws_permute)
    L.y_perm.fill_(float("nan"))
    call(cfg, x, L.perm, L.offsets, *q, L.y_perm, L.ws_ffn)
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


@pytest.mark.parametrize("kind", ["fp8", "mxfp4"])
@pytest.mark.parametrize("counts,d,d_ff", SPLIT)
def test_split_kernel_edges(kind, counts, d, d_ff):
    eidx = np.random.default_rng(5).permutation(np.repeat(np.arange(4), counts)).astype(np.int32).reshape(-1, 1)
    print(f"[q split] {kind} counts={counts} d={d} d_ff={d_ff}", flush=True)
    _check(kind, sum(counts), d, 2, d_ff, eidx)


@pytest.mark.parametrize("kind,d,n,d_ff", STAGED)
def test_staged_kernel(kind, d, n, d_ff):
    T, rng = 32, np.random.default_rng(7)
    waves = min(2 * T, 2 * n) * (sum(d_ff) // 2) // 16
    assert waves >= (6500 if kind == "fp8" else 3000) and (kind == "fp8" or not any(f % 128 for f in d_ff)), "a shape for the split kernel"
    eidx = np.stack([rng.integers(0, n, T), n + rng.integers(0, n, T)], 1).astype(np.int32)
    print(f"[q staged] {kind} d={d} waves={waves}", flush=True)
    _check(kind, T, d, n, d_ff, eidx)
