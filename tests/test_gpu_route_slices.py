"""The router at hidden sizes that its waves and workgroups cannot share evenly, against float64."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _check(d, dtype, ng, n, tokens):
    import paper_2604_23108_amd as M
    kg, ke = 2, 4
    gen = torch.Generator(device="cuda").manual_seed(d)
    wg, we = (torch.randn((r, d), generator=gen, device="cuda") * 0.05 for r in (ng, ng * n))
    for T in tokens:
        x = torch.randn((T, d), generator=gen, device="cuda")
        x = x.bfloat16() if dtype == "bf16" else x
        cfg = M.Config(T=T, d=d, n_groups=ng, experts_per_group=n, d_ff=(64,) * ng, k_groups=kg, k_experts=ke,
                       select_mode=M.SELECT_GLOBAL, dtype=M.BF16 if dtype == "bf16" else M.F32)
        new = lambda k, t: torch.full((T, k), -1, dtype=t, device="cuda")
        gi, ei, gates = new(kg, torch.int32), new(ke, torch.int32), new(ke, torch.float32)
        nb = M.mohge_workspace_size(cfg, M.CALL_ROUTE)
        ws = torch.empty(nb, dtype=torch.uint8, device="cuda") if nb else None
        print(f"[route] d={d} T={T} {dtype}", flush=True)
        M.mohge_route(cfg, x, wg, we, None, gi, ei, gates, None, None, ws)
        X = x.double()
        zg, ze = X @ wg.double().T.contiguous(), X @ we.double().T.contiguous()
        kept = zg.gather(1, gi.long())
        out = zg.scatter(1, gi.long(), float("-inf"))
        assert (kept.min(1).values >= out.max(1).values - 1e-6).all()      # margins below the error of a logit are ties
        e2 = torch.softmax(ze.view(T, ng, n), -1) * torch.sigmoid(zg)[:, :, None]
        mask = torch.zeros_like(zg).scatter(1, gi.long(), 1.0)
        e2 = (e2 * mask[:, :, None]).view(T, -1)
        sel = e2.gather(1, ei.long())
        assert (sel.min(1).values >= e2.scatter(1, ei.long(), -1.0).max(1).values - 1e-6).all()
        assert (ei[:, 1:] > ei[:, :-1]).all()
        # gates: fp32 logits to about 1e-7, expf to about an ulp
        assert (gates.double() - sel / sel.sum(1, keepdim=True)).abs().max() <= 1e-6


@pytest.mark.parametrize("d", [64, 128, 192, 704, 1344, 2624])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_route_uneven_slices(d, dtype):
    _check(d, dtype, 5, 5, (1, 17, 300, 2049, 4100))


@pytest.mark.parametrize("ng,n", [(2, 4), (3, 8), (5, 7), (4, 12), (2, 32), (8, 16)])
@pytest.mark.parametrize("d", [128, 384, 640, 1152])
def test_route_many_tokens(d, ng, n):
    """One to five and more column tiles of router rows, one chunk of the hidden dimension to several groups of them, 32 and 64
    tokens per workgroup, more workgroups than compute units; selection inside the logits kernel and in a second one."""
    _check(d, "bf16", ng, n, (4097, 8192, 8193, 12800, 16400))


@pytest.mark.parametrize("ng,n", [(2, 4), (3, 8), (5, 7)])
def test_route_many_tokens_deep(ng, n):
    """Long reductions, where one to three column tiles go to a second kernel too."""
    _check(4096, "bf16", ng, n, (4097, 8192, 8193, 16400))


@pytest.mark.parametrize("T", [300, 4100, 8200])
@pytest.mark.parametrize("sign", [-1, 1])
def test_route_infinite_weight(T, sign):
    """A router weight of -inf times positive elements is a logit of -inf, in every form: the expert is as if its bias were -inf.
    (+inf: the group's softmax is NaN, as it is in the fp32 form, and every id is still one of an expert.)"""
    import paper_2604_23108_amd as M
    d, ng, n, kg, ke = 256, 8, 4, 3, 6
    gen = torch.Generator(device="cuda").manual_seed(T)
    wg, we = (torch.randn((r, d), generator=gen, device="cuda") * 0.1 for r in (ng, ng * n))
    x = torch.randn((T, d), generator=gen, device="cuda")
    x[:, 5] = x[:, 5].abs() + 0.5
    x = x.bfloat16()
    cfg = M.Config(T=T, d=d, n_groups=ng, experts_per_group=n, d_ff=(64,) * ng, k_groups=kg, k_experts=ke,
                   select_mode=M.SELECT_GLOBAL, dtype=M.BF16)
    size = M.mohge_workspace_size(cfg, M.CALL_ROUTE)

    def call(w, bias):
        i32 = dict(dtype=torch.int32, device="cuda")
        f32 = dict(dtype=torch.float32, device="cuda")
        out = (torch.full((T, kg), -1, **i32), torch.full((T, ke), -1, **i32), torch.zeros((T, ke), **f32),
               torch.zeros((T, ng), **f32), torch.zeros((T, ng * n), **f32))
        M.mohge_route(cfg, x, wg, w, bias, *out, torch.empty(size, dtype=torch.uint8, device="cuda") if size else None)
        return out

    inf = float("inf") * sign
    weight, bias = we.clone(), torch.zeros(ng * n, device="cuda")
    weight[13, 5], bias[13] = inf, inf
    got, want = call(weight, None), call(we, bias)
    assert ((got[1] >= 0) & (got[1] < ng * n)).all() and ((got[0] >= 0) & (got[0] < ng)).all()
    for a, b in zip(got, want):
        assert torch.equal(torch.nan_to_num(a.float(), nan=-7.0), torch.nan_to_num(b.float(), nan=-7.0))
    if sign < 0:
        assert not (got[1] == 13).any() and all(torch.isfinite(t.float()).all() for t in got)
