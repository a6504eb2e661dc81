"""The fp32 expert networks at the edges of their tiles (32 token rows, 64 weight rows, 64-deep
stages), on a hand-made assignment of tokens to experts, against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
from synth import Workload, generate

pytestmark = pytest.mark.gpu

# rows per expert: none, one, around one, two and several tiles
COUNTS = [0, 1, 31, 32, 33, 63, 64, 65, 97, 130, 0, 200]


@pytest.mark.parametrize("d,d_ff", [(64, (64, 128)), (192, (320, 64)), (1024, (192, 448))])
def test_ffn_f32_tile_edges(d, d_ff):
    import paper_2604_23108_amd as M
    from gpu_harness import DeviceLayer
    T = sum(COUNTS)                                     # one pair per token: any assignment is possible
    w = Workload("f32_edges", T=T, d=d, n_groups=2, experts_per_group=6, d_ff=d_ff, k_groups=1, k_experts=1,
                 dtype="f32", seed=41)
    inp = generate(w)
    dl = DeviceLayer(w, inp, training=False, guard=True)
    L = dl.layer
    eidx = np.random.default_rng(5).permutation(np.repeat(np.arange(12), COUNTS)).astype(np.int32).reshape(T, 1)
    M.mohge_permute(dl.cfg, torch.from_numpy(eidx).cuda(), L.counts, L.offsets, L.perm, L.inv_perm, None, None,
                    L.ws_permute)
    L.y_perm.fill_(float("nan"))
    print(f"[f32 edges] d={d} d_ff={d_ff}", flush=True)
    M.mohge_expert_ffn(dl.cfg, dl.x, L.perm, L.offsets, L.w13, L.w2, L.y_perm, L.ws_ffn)
    dl.check_guards()
    want = oracle.expert_ffn(w, inp.x.f32, [t.f32 for t in inp.w_gate], [t.f32 for t in inp.w_up],
                             [t.f32 for t in inp.w_down], np.arange(T, dtype=np.int32), eidx.reshape(-1))
    got = L.y_perm.cpu().numpy()
    want = want[L.perm.cpu().numpy()]
    # two fp32 dot products in chains of 8 with fp64 totals and the roundings between them: relative to the largest
    # output the error stays below 2^-24 * (8 + 16) with room to spare
    assert np.isfinite(got).all()
    assert np.abs(got - want).max() <= 5e-6 * np.abs(want).max()


@pytest.mark.parametrize("d,d_ff", [(64, (64, 128)), (128, (64, 256)), (512, (256, 448)), (1024, (192, 896)),
                                    (4096, (768, 2048))])
def test_ffn_f32_rounding_error(d, d_ff):
    """Error of the fp32 expert networks against float64, as a 2-norm.  A rounding costs 2.5e-8 rms
    (2^-24 / sqrt(3), averaged over the mantissa).  A dot product in chains of eight products, added in pairs to an
    fp64 total, carries the roundings of 4.5 + 1 + 1 of its values: 6.4e-8, whatever its length.  Both operands of
    SiLU(a) b have it, the first amplified by up to 1.5, SiLU and the product add about four roundings, the second
    projection its own: sqrt(6.4^2 (1 + 1.5^2) + 4 * 2.5^2 + 6.4^2) = 14e-8."""
    import paper_2604_23108_amd as M
    from gpu_harness import DeviceLayer
    T, n = 128, 2
    w = Workload("f32_err", T=T, d=d, n_groups=2, experts_per_group=n, d_ff=d_ff, k_groups=1, k_experts=1,
                 dtype="f32", seed=44)
    dl = DeviceLayer(w, generate(w), training=False)
    L = dl.layer
    eidx = np.repeat(np.arange(4), T // 4).astype(np.int32).reshape(T, 1)
    M.mohge_permute(dl.cfg, torch.from_numpy(eidx).cuda(), L.counts, L.offsets, L.perm, L.inv_perm, None, None,
                    L.ws_permute)
    print(f"[f32 error] d={d} d_ff={d_ff}", flush=True)
    M.mohge_expert_ffn(dl.cfg, dl.x, L.perm, L.offsets, L.w13, L.w2, L.y_perm, L.ws_ffn)
    torch.cuda.synchronize()
    rows = dl.x[L.perm.long()].cpu().double().view(4, T // 4, d)
    want = []
    for e in range(4):
        g, i = divmod(e, n)
        w13, w2 = L.w13[g][i].cpu().double(), L.w2[g][i].cpu().double()
        a, b = (rows[e] @ w13.T).split(d_ff[g], dim=1)
        want.append((a * torch.sigmoid(a) * b) @ w2.T)
    want = torch.cat(want)
    err = float((L.y_perm.cpu().double() - want).norm() / want.norm())
    assert err <= 1.5e-7, err


def test_ffn_f32_operands_without_a_finite_bf16_part():
    """Operands near the largest fp32 number (infinity in bf16), infinities and NaN: sums that are finite come out as such, and
    the rows beside those that are not stay as they are."""
    import paper_2604_23108_amd as M
    T, d, F = 6, 192, 64
    cfg = M.Config(T=T, d=d, n_groups=1, experts_per_group=1, d_ff=(F,), k_groups=1, k_experts=1,
                   select_mode=M.SELECT_PER_GROUP, dtype=M.F32)
    gen = torch.Generator().manual_seed(9)
    x = torch.randn((T, d), generator=gen)
    w13, w2 = torch.randn((1, 2 * F, d), generator=gen) * 0.1, torch.randn((1, d, F), generator=gen) * 0.1
    w13[0, :, 70] *= 1e-37
    x[1, 5], x[2, 150], x[3, 70], x[4] = float("inf"), float("nan"), 3.4e38, x[4] * 2.0 ** 55
    a, b = (x.double() @ w13[0].double().T).split(F, dim=1)
    want = (a * torch.sigmoid(a) * b) @ w2[0].double().T
    offsets = torch.tensor([0, T], dtype=torch.int32, device="cuda")
    y = torch.zeros((T, d), device="cuda")
    ws = torch.empty(M.mohge_workspace_size(cfg, M.CALL_EXPERT_FFN), dtype=torch.uint8, device="cuda")
    print("[f32 extremes]", flush=True)
    M.mohge_expert_ffn(cfg, x.cuda(), None, offsets, [w13.cuda()], [w2.cuda()], y, ws)
    y = y.cpu().double()
    assert not torch.isfinite(y[1:3]).any()
    for t in (0, 3, 4, 5):
        # the bound of the error test above, per row of 192 values instead of over all of them
        assert float((y[t] - want[t]).norm() / want[t].norm()) <= 3e-7, t


def _second_projection(h, w2):
    """The second projection alone: y = h . w2^T in fp32 and in float64."""
    import paper_2604_23108_amd as M
    (T, K), d = h.shape, w2.shape[1]
    cfg = M.Config(T=T, d=d, n_groups=1, experts_per_group=1, d_ff=(K,), k_groups=1, k_experts=1,
                   select_mode=M.SELECT_PER_GROUP, dtype=M.F32)
    y = torch.full((T, d), float("nan"), device="cuda")
    M.mohge_expert_ffn_down(cfg, h.cuda(), torch.tensor([0, T], dtype=torch.int32, device="cuda"), [w2.cuda()], y)
    return y.cpu().double(), h.double() @ w2[0].double().T


@pytest.mark.parametrize("K", [256, 4096, 16384])
def test_ffn_f32_outlier_channels(K):
    """A few channels a thousand times as large as the others: most products are added to a sum that is much larger.  Sums
    that round to nearest are off by 6.5 roundings (6.4e-8, see above) at any length and to both sides alike; units that
    cut off what lies below the sum drift to one side, in proportion to the length."""
    gen = torch.Generator().manual_seed(K)
    h, w2 = torch.randn((96, K), generator=gen), torch.randn((1, 320, K), generator=gen)
    h[:, ::97] *= 1000.0
    print(f"[f32 outliers] K={K}", flush=True)
    y, want = _second_projection(h, w2)
    err = y - want
    # 30720 outputs: the mean of errors without a drift is below 4 / sqrt(30720) = 0.023 of their mean size
    assert abs(float(err.mean() / err.abs().mean())) <= 0.05
    # (a chain holds one outlier or none at the short length, and the sum of the few there are rounds once more)
    assert float(err.norm() / want.norm()) <= (7.5e-8 if K > 1024 else 9e-8)


@pytest.mark.parametrize("lo,hi", [(-112, 100), (-118, 110), (-125, 118)])
def test_ffn_f32_operands_near_the_smallest_normal_number(lo, hi):
    """Very small operands of one side times very large ones of the other give ordinary sums: every bit of the small ones
    counts, down to the smallest normal number (2^-126; smaller ones have fewer bits to begin with)."""
    gen = torch.Generator().manual_seed(-lo)
    small, large = [(1.0 + torch.rand(s, generator=gen)) * torch.randint(0, 2, s, generator=gen).mul(2).sub(1) * 2.0 ** k
                    for s, k in (((64, 256), lo), ((1, 192, 256), hi))]
    print(f"[f32 small] 2^{lo} x 2^{hi}", flush=True)
    for h, w2 in ((small, large), (large[0], small.unsqueeze(0))):
        y, want = _second_projection(h, w2)
        # 6.5 roundings as above (6.4e-8)
        assert float((y - want).norm() / want.norm()) <= 7.5e-8


def test_ffn_f32_more_workgroups_than_one_grid_dimension():
    """2^20 routed rows of an expert 16384 wide: 2^24 workgroups of the first projection, whose threads do not fit one
    dimension of a grid (64 GiB of hidden activations).  Rows repeat with a period of 4096, results have to as well."""
    import paper_2604_23108_amd as M
    T, d, F, period = 1 << 20, 64, 1 << 14, 4096
    cfg = M.Config(T=T, d=d, n_groups=1, experts_per_group=1, d_ff=(F,), k_groups=1, k_experts=1,
                   select_mode=M.SELECT_PER_GROUP, dtype=M.F32)
    need = M.mohge_workspace_size(cfg, M.CALL_EXPERT_FFN)
    assert need == T * F * 4
    if torch.cuda.mem_get_info()[0] < need + (4 << 30):
        pytest.skip("needs 68 GiB of free device memory")
    gen = torch.Generator(device="cuda").manual_seed(3)
    normal = lambda *s: torch.randn(s, generator=gen, device="cuda")
    x = normal(period, d)
    w13, w2 = normal(1, 2 * F, d) * 0.1, normal(1, d, F) * 0.02
    offsets = torch.tensor([0, T], dtype=torch.int32, device="cuda")
    y = torch.full((T, d), float("nan"), device="cuda")
    print(f"[f32 grid] rows={T} width={F}", flush=True)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    M.mohge_expert_ffn(cfg, x.repeat(T // period, 1), None, offsets, [w13], [w2], y, ws)
    torch.cuda.synchronize()
    del ws
    y = y.view(T // period, period, d)
    assert torch.equal(y, y[:1].expand_as(y))
    a, b = (x.double() @ w13[0].double().T.contiguous()).split(F, dim=1)
    want = (a * torch.sigmoid(a) * b) @ w2[0].double().T.contiguous()
    # the bound of the error test above
    assert float((y[0].double() - want).norm() / want.norm()) <= 1.5e-7
    torch.cuda.empty_cache()


@pytest.mark.parametrize("d,d_ff", [(64, (64, 128)), (192, (320, 64)), (1024, (192, 448))])
def test_ffn_f32_half_tiles(d, d_ff):
    """Row tiles of at most 16 rows have MFMAs of their own: experts whose last tile is around that size, alone and behind whole
    tiles.  Their sums are in groups of eight products as well, so the bound of test_ffn_f32_rounding_error holds for them: here for
    the rows of these tiles alone."""
    import paper_2604_23108_amd as M
    from gpu_harness import DeviceLayer
    counts = [15, 16, 17, 47, 48, 49, 2, 0, 9, 80, 1, 31]
    T, n = sum(counts), 6
    w = Workload("f32_half", T=T, d=d, n_groups=2, experts_per_group=n, d_ff=d_ff, k_groups=1, k_experts=1, dtype="f32", seed=47)
    dl = DeviceLayer(w, generate(w), training=False, guard=True)
    L = dl.layer
    eidx = np.random.default_rng(6).permutation(np.repeat(np.arange(2 * n), counts)).astype(np.int32).reshape(T, 1)
    M.mohge_permute(dl.cfg, torch.from_numpy(eidx).cuda(), L.counts, L.offsets, L.perm, L.inv_perm, None, None,
                    L.ws_permute)
    L.y_perm.fill_(float("nan"))
    print(f"[f32 half tiles] d={d} d_ff={d_ff}", flush=True)
    M.mohge_expert_ffn(dl.cfg, dl.x, L.perm, L.offsets, L.w13, L.w2, L.y_perm, L.ws_ffn)
    dl.check_guards()
    rows = dl.x[L.perm.long()].cpu().double()
    y = L.y_perm.cpu().double()
    at, off, norm = 0, 0.0, 0.0
    for e, c in enumerate(counts):
        g, i = divmod(e, n)
        w13, w2 = L.w13[g][i].cpu().double(), L.w2[g][i].cpu().double()
        a, b = (rows[at:at + c] @ w13.T).split(d_ff[g], dim=1)
        want, got = (a * torch.sigmoid(a) * b) @ w2.T, y[at:at + c]
        assert torch.isfinite(got).all()
        if c:
            assert float((got - want).abs().max()) <= 5e-6 * float(want.abs().max()), e      # as in the test of the tile edges
            if 0 < c % 32 <= 16:
                last = slice(c - c % 32, c)
                off, norm = off + float((got - want)[last].square().sum()), norm + float(want[last].square().sum())
        at += c
    assert (off / norm) ** 0.5 <= 1.5e-7


@pytest.mark.parametrize("d,F", [(64, 64), (192, 320), (1024, 896)])
def test_ffn_f32_a_row_does_not_depend_on_its_tile(d, F):
    """The result of a row is the same, bit for bit, whether the rows around it fill a tile of 32 or leave it with 16 or fewer:
    both kinds of tile add up the same groups of eight products in the same order."""
    import paper_2604_23108_amd as M
    gen = torch.Generator().manual_seed(d + F)
    x = torch.randn((64, d), generator=gen).cuda()
    w13, w2 = (torch.randn((1, 2 * F, d), generator=gen) * 0.1).cuda(), (torch.randn((1, d, F), generator=gen) * 0.1).cuda()

    def layer(T):
        cfg = M.Config(T=T, d=d, n_groups=1, experts_per_group=1, d_ff=(F,), k_groups=1, k_experts=1,
                       select_mode=M.SELECT_PER_GROUP, dtype=M.F32)
        y = torch.full((T, d), float("nan"), device="cuda")
        ws = torch.empty(M.mohge_workspace_size(cfg, M.CALL_EXPERT_FFN), dtype=torch.uint8, device="cuda")
        M.mohge_expert_ffn(cfg, x[:T].contiguous(), None, torch.tensor([0, T], dtype=torch.int32, device="cuda"), [w13], [w2], y, ws)
        return y.cpu()

    print(f"[f32 tile of a row] d={d} F={F}", flush=True)
    want = layer(64)
    assert torch.isfinite(want).all()
    for T in (1, 7, 15, 16, 17, 32, 33, 47, 48, 49):
        assert torch.equal(layer(T), want[:T]), T
