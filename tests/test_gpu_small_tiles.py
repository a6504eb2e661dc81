"""The 128 x 128 tile form of the bf16 expert networks at the edges of its tiles, forward and backward,
bit by bit against the 256 x 256 form (both add the products of an output in the same order) and, forward,
against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
from synth import Workload, generate

pytestmark = pytest.mark.gpu

# rows per expert: none, one, around one fragment, one tile, several tiles and one band of four
COUNTS = [0, 1, 31, 64, 65, 127, 128, 129, 0, 257, 513, 640]


@pytest.mark.parametrize("d,d_ff", [(64, (64, 128)), (192, (320, 64)), (1024, (192, 448))])
def test_small_tiles_equal_big_tiles(d, d_ff):
    import paper_2604_23108_amd as M
    from paper_2604_23108_amd import bench_binding as BB
    from gpu_harness import DeviceLayer, to_dev
    T = sum(COUNTS)                                     # one pair per token: any assignment is possible
    w = Workload("small_tiles", T=T, d=d, n_groups=2, experts_per_group=6, d_ff=d_ff, k_groups=1, k_experts=1,
                 seed=43, training=True)
    inp = generate(w)
    dl = DeviceLayer(w, inp, backward=True, guard=True)
    L = dl.layer
    eidx = np.random.default_rng(5).permutation(np.repeat(np.arange(12), COUNTS)).astype(np.int32).reshape(T, 1)
    M.mohge_permute(dl.cfg, torch.from_numpy(eidx).cuda(), L.counts, L.offsets, L.perm, L.inv_perm, None, None,
                    L.ws_permute)
    L.dy_perm.copy_(to_dev(inp.dy, True)[L.perm.long()])
    outs = []
    for form in ("by size", "small", "big"):
        for t in [L.y_perm, L.dx_perm, *L.dw13, *L.dw2]:
            t.fill_(float("nan"))
        print(f"[small tiles] d={d} d_ff={d_ff} form={form}", flush=True)
        args = (dl.cfg, dl.x, L.perm, L.offsets, L.w13, L.w2)
        if form == "by size":
            M.mohge_expert_ffn(*args, L.y_perm, L.ws_ffn)
            y = L.y_perm.clone()
            M.mohge_expert_ffn_train(*args, L.y_perm, L.saved)
            M.mohge_expert_ffn_bwd(*args, L.saved, L.dy_perm, L.dx_perm, L.dw13, L.dw2, L.ws_ffn_bwd)
            for call, ws in ((M.CALL_EXPERT_FFN, L.ws_ffn), (M.CALL_FFN_SAVED, L.saved), (M.CALL_EXPERT_FFN_BWD, L.ws_ffn_bwd)):
                assert M.mohge_fused_status(dl.cfg, call, ws) == 0
        else:
            o = BB.FfnOptions(small_tiles=int(form == "small"))
            BB.mohge_bench_expert_ffn(*args, L.y_perm, L.ws_ffn, o)
            y = L.y_perm.clone()
            BB.mohge_bench_expert_ffn_train(*args, L.y_perm, L.saved, o)
            BB.mohge_bench_expert_ffn_bwd(*args, L.saved, L.dy_perm, L.dx_perm, L.dw13, L.dw2, L.ws_ffn_bwd, o)
        torch.cuda.synchronize()
        dl.check_guards()
        outs.append([t.clone().view(torch.int16) for t in [y, L.y_perm, L.dx_perm, *L.dw13, *L.dw2]])
    for a, b, c in zip(*outs):
        assert torch.equal(a, b) and torch.equal(b, c)
    want = oracle.expert_ffn(w, inp.x.f32, [t.f32 for t in inp.w_gate], [t.f32 for t in inp.w_up],
                             [t.f32 for t in inp.w_down], np.arange(T, dtype=np.int32), eidx.reshape(-1))
    got, want = L.y_perm.float().cpu().numpy(), want[L.perm.cpu().numpy()]
    # h and y are rounded to bf16 once each: 2^-9 of the value and of a sum of such terms
    assert np.abs(got - want).max() <= 8e-3 * np.abs(want).max()


# rows per expert where most experts are one tall tile: its edges, and one expert of each other kind; too few for it
TALL = [129, 192, 191, 160, 130, 161, 144, 180, 128, 193, 150, 190]
FEW_TALL = [129, 192, 191, 64, 130, 161, 65, 257, 128, 193, 150, 320]


def _tall_equals_big(d, d_ff, per_group, counts, permuted=True):
    import paper_2604_23108_amd as M
    from paper_2604_23108_amd import bench_binding as BB
    from gpu_harness import DeviceLayer, to_dev
    T, ne = sum(counts), len(counts)
    assert 140 * ne <= T <= 184 * ne
    w = Workload("tall_tiles", T=T, d=d, n_groups=2, experts_per_group=per_group, d_ff=d_ff, k_groups=1, k_experts=1, seed=47,
                 training=True)
    inp = generate(w)
    dl = DeviceLayer(w, inp, backward=True, guard=True)
    L = dl.layer
    eidx = np.random.default_rng(6).permutation(np.repeat(np.arange(ne), counts)).astype(np.int32).reshape(T, 1)
    M.mohge_permute(dl.cfg, torch.from_numpy(eidx).cuda(), L.counts, L.offsets, L.perm, L.inv_perm, None, None,
                    L.ws_permute)
    L.dy_perm.copy_(to_dev(inp.dy, True)[L.perm.long()])
    x, perm = (dl.x, L.perm) if permuted else (dl.x[L.perm.long()].contiguous(), None)
    outs = []
    for small in (1, 0):
        for t in [L.y_perm, L.dx_perm, *L.dw13, *L.dw2]:
            t.fill_(float("nan"))
        print(f"[tall tiles] d={d} d_ff={d_ff} experts={ne} permuted={permuted} small={small}", flush=True)
        args, o = (dl.cfg, x, perm, L.offsets, L.w13, L.w2), BB.FfnOptions(small_tiles=small)
        BB.mohge_bench_expert_ffn(*args, L.y_perm, L.ws_ffn, o)
        y = L.y_perm.clone()
        BB.mohge_bench_expert_ffn_train(*args, L.y_perm, L.saved, o)
        BB.mohge_bench_expert_ffn_bwd(*args, L.saved, L.dy_perm, L.dx_perm, L.dw13, L.dw2, L.ws_ffn_bwd, o)
        torch.cuda.synchronize()
        dl.check_guards()
        outs.append([t.clone() for t in [y, L.y_perm, L.dx_perm, *L.dw13, *L.dw2]])
    for a, b in zip(*outs):
        assert torch.isfinite(a.float()).all() and torch.equal(a, b)


@pytest.mark.parametrize("counts", [TALL, FEW_TALL], ids=["tall", "few"])
@pytest.mark.parametrize("d,d_ff", [(64, (64, 128)), (192, (320, 64)), (1024, (192, 448)), (2816, (128, 320))])
def test_tall_tiles_equal_big_tiles(d, d_ff, counts):
    """Bit by bit: every output adds its products in the same order in either form.  (Few tiles: of the launches only dX takes tall
    ones, at d = 2816.)"""
    _tall_equals_big(d, d_ff, 6, counts)


def _tiles(counts, columns, tall):
    """row tiles of 128, or one of 192 for 129 to 192 rows, times the column tiles of the expert's group"""
    half = len(counts) // 2
    return sum((1 if tall and 128 < c <= 192 else -(-c // 128)) * columns[i // half] for i, c in enumerate(counts))


@pytest.mark.parametrize("permuted", [True, False])
@pytest.mark.parametrize("per_group,d,d_ff,launches", [(36, 1024, (384, 320), "up down dH dX"), (33, 1088, (384, 448), "up down dH dX"),
                                                       (32, 1024, (320, 448), "up down dH dX"), (36, 64, (384, 320), "up dH"),
                                                       (12, 2048, (960, 1024), "up dH dX"), (36, 1024, (384, 320), "")])
def test_tall_tiles_by_launch(per_group, d, d_ff, launches, permuted):
    """Most of 24 to 72 experts tall, the others in the first and the last ones of the list: with more than 64 of them the list
    has two rounds.  Sizes at which the launches named take tall tiles (256 compute units); d = 64: a reduction of one stage.  Last:
    too few experts of that size.  Rows given in expert order as well."""
    rng = np.random.default_rng(per_group)
    counts = [int(c) for c in rng.integers(129, 193, 2 * per_group)]
    counts[:9] = [129, 0, 192, 191, 130, 160, 161, 128, 129]
    if per_group > 12:
        counts[per_group - 1], counts[-2], counts[-1] = 192, 257, 64
    if not launches:
        counts[10:30] = [128, 200] * 10
    few = 4 * sum(128 < c <= 192 for c in counts) < 3 * len(counts)
    assert few == (not launches)
    assert 20 * sum(c > 192 for c in counts) <= len(counts) or few
    for name, columns, lo, hi in (("up", [-(-f // 64) for f in d_ff], 192, 512), ("down", [-(-d // 128)] * 2, 512, 1 << 30),
                                  ("dH", [-(-f // 128) for f in d_ff], 180, 512), ("dX", [-(-d // 128)] * 2, 192, 1 << 30)):
        takes = lo <= per_group * sum(columns) <= hi and _tiles(counts, columns, True) <= hi and not few
        assert takes == (name in launches.split()), name
    _tall_equals_big(d, d_ff, per_group, counts, permuted)


@pytest.mark.parametrize("forward,backward", [(1, 0), (0, 1)])
def test_forward_and_backward_in_different_forms(forward, backward):
    """The two rules differ, so a layer may run its forward in small tiles and its backward in big ones: what the forward
    keeps is the same in either form."""
    from paper_2604_23108_amd import bench_binding as BB
    from gpu_harness import DeviceLayer, to_dev
    w = Workload("mixed_forms", T=333, d=192, n_groups=2, experts_per_group=4, d_ff=(320, 64), k_groups=2, k_experts=4,
                 seed=59, training=True)
    inp = generate(w)
    dl = DeviceLayer(w, inp, backward=True, guard=True)
    L, dy = dl.layer, to_dev(inp.dy, True)
    outs = []
    for f, b in ((forward, backward), (0, 0)):
        for t in [L.y, L.dx, L.dx_perm, *L.dw13, *L.dw2]:
            t.fill_(float("nan"))
        L.saved.fill_(0xFF)
        print(f"[mixed forms] forward small={f} backward small={b}", flush=True)
        L.ffn_options = BB.FfnOptions(small_tiles=f)
        L.forward(dl.x)
        L.ffn_options = BB.FfnOptions(small_tiles=b)
        L.backward(dl.x, dy)
        torch.cuda.synchronize()
        dl.check_guards()
        outs.append([t.clone() for t in [L.y, L.dx, *L.dw13, *L.dw2, L.dw_expert]])
    for a, b in zip(*outs):
        assert torch.isfinite(a.float()).all() and torch.equal(a, b)


@pytest.mark.parametrize("with_perm", [True, False])
def test_backward_of_a_call_without_tokens(with_perm):
    """T = 0 is a valid call: the weight gradients are sums over no rows, zeros."""
    import paper_2604_23108_amd as M
    d, ff, n = 192, (64, 128), 3
    cfg = M.Config(T=0, d=d, n_groups=2, experts_per_group=n, d_ff=ff, k_groups=1, k_experts=1,
                   select_mode=M.SELECT_PER_GROUP, dtype=M.BF16)
    bf = dict(dtype=torch.bfloat16, device="cuda")
    row = lambda: torch.full((16, d), float("nan"), **bf)              # never read or written
    perm = torch.full((16,), -1, dtype=torch.int32, device="cuda")
    offsets = torch.zeros(2 * n + 1, dtype=torch.int32, device="cuda")
    w13, w2 = [torch.ones((n, 2 * f, d), **bf) for f in ff], [torch.ones((n, d, f), **bf) for f in ff]
    dw13, dw2 = [torch.full_like(w, float("nan")) for w in w13], [torch.full_like(w, float("nan")) for w in w2]
    u8 = lambda call: torch.full((M.mohge_workspace_size(cfg, call),), 0xFF, dtype=torch.uint8, device="cuda")
    dx_perm = row()
    print(f"[no tokens] perm={with_perm}", flush=True)
    M.mohge_expert_ffn_bwd(cfg, row(), perm if with_perm else None, offsets, w13, w2, u8(M.CALL_FFN_SAVED), row(), dx_perm,
                           dw13, dw2, u8(M.CALL_EXPERT_FFN_BWD))
    torch.cuda.synchronize()
    for t in dw13 + dw2:
        assert not t.any()
    assert torch.isnan(dx_perm.float()).all()


def test_small_tiles_leave_the_clock_counters_alone():
    """The counters have room for a workgroup per compute unit; the small form has more, and counts nothing: neither in the buffer
    nor behind it."""
    import paper_2604_23108_amd as M
    from paper_2604_23108_amd import bench_binding as BB
    from gpu_harness import DeviceLayer, to_dev
    w = Workload("small_cycles", T=900, d=512, n_groups=2, experts_per_group=8, d_ff=(512, 1024), k_groups=1, k_experts=2,
                 seed=48, training=True)
    inp = generate(w)
    dl = DeviceLayer(w, inp, backward=True)
    dl.run()
    L = dl.layer
    L.dy_perm.copy_(to_dev(inp.dy, True)[(L.perm // 2).long()])
    room = BB.cycles_buffer()
    buf = torch.zeros((64,) + tuple(room.shape), dtype=torch.int64, device="cuda")      # (64 times the room for what came behind it)
    print("[small tiles] clock counters", flush=True)
    args = (dl.cfg, dl.x, L.perm, L.offsets, L.w13, L.w2)
    for launch in (0, 1):
        o = BB.FfnOptions(cycles=buf[0], cycles_launch=launch, small_tiles=1)
        BB.mohge_bench_expert_ffn(*args, L.y_perm, L.ws_ffn, o)
        BB.mohge_bench_expert_ffn_train(*args, L.y_perm, L.saved, o)
        BB.mohge_bench_expert_ffn_bwd(*args, L.saved, L.dy_perm, L.dx_perm, L.dw13, L.dw2, L.ws_ffn_bwd, o)
    torch.cuda.synchronize()
    assert int(buf.abs().sum()) == 0
    o = BB.FfnOptions(cycles=buf[0], small_tiles=0)
    BB.mohge_bench_expert_ffn(*args, L.y_perm, L.ws_ffn, o)
    torch.cuda.synchronize()
    assert int(buf[0, 0, :, 4].sum()) > 0 and int(buf[1:].abs().sum()) == 0
