"""bf16 expert networks whose weight rows are so long that the rows of one tile span more than 4 GiB."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,F", [((1 << 24) + (1 << 20), 128), (256, (1 << 23) + (1 << 19))], ids=["first", "second"])
def test_ffn_rows_of_a_tile_span_more_than_4_gib(d, F):
    """One expert, weights that are zero but for 96 reduction indices spread over the rows; by itself, and captured and replayed."""
    import paper_2604_23108_amd as M
    T, K = 200, max(d, F)
    if torch.cuda.mem_get_info()[0] < 8 * (T + 3 * min(d, F)) * K:
        pytest.skip("needs up to 100 GiB of free device memory")
    cfg = M.Config(T=T, d=d, n_groups=1, experts_per_group=1, d_ff=(F,), k_groups=1, k_experts=1,
                   select_mode=M.SELECT_PER_GROUP, dtype=M.BF16)
    gen = torch.Generator(device="cuda").manual_seed(7)
    normal = lambda *s: torch.randn(s, generator=gen, device="cuda").to(torch.bfloat16)
    idx = torch.cat([torch.arange(0, 32), torch.randint(0, K, (32,), generator=torch.Generator().manual_seed(1)),
                     torch.arange(K - 32, K)]).unique().cuda()
    x, w13, w2 = (torch.zeros(s, dtype=torch.bfloat16, device="cuda") for s in ((T, d), (1, 2 * F, d), (1, d, F)))
    if d == K:
        x[:, idx], w13[0, :, idx], w2[0] = normal(T, len(idx)), normal(2 * F, len(idx)) * 0.1, normal(d, F) * 0.1
    else:
        both = torch.cat([idx, idx + F])
        x.copy_(normal(T, d))
        w13[0, both], w2[0, :, idx] = normal(len(both), d) * 0.1, normal(d, len(idx)) * 0.1
    offsets = torch.tensor([0, T], dtype=torch.int32, device="cuda")
    y = torch.full((T, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(M.mohge_workspace_size(cfg, M.CALL_EXPERT_FFN), dtype=torch.uint8, device="cuda")
    print(f"[long rows] d={d} F={F}", flush=True)
    M.mohge_expert_ffn(cfg, x, None, offsets, [w13], [w2], y, ws)
    assert M.mohge_fused_status(cfg, M.CALL_EXPERT_FFN, ws) == 0
    bits = y.clone()
    y.fill_(float("nan"))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        M.mohge_expert_ffn(cfg, x, None, offsets, [w13], [w2], y, ws)
    for _ in range(3):
        y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y.view(torch.int16), bits.view(torch.int16))
    del graph, bits
    if d == K:
        a, b = (x[:, idx].float() @ w13[0][:, idx].float().T.contiguous()).split(F, dim=1)
        cols = idx
        h = (a * torch.sigmoid(a) * b).to(torch.bfloat16)
        want = h.float() @ w2[0][cols].float().T.contiguous()
    else:
        cols = torch.arange(d, device="cuda")
        a, b = (x.float() @ w13[0][idx].float().T.contiguous()), (x.float() @ w13[0][idx + F].float().T.contiguous())
        h = (a * torch.sigmoid(a) * b).to(torch.bfloat16)
        want = h.float() @ w2[0][:, idx].float().T.contiguous()
    got = y[:, cols].float()
    # h and y are rounded to bf16 (2^-9 each at most, about half of that in the mean); a value of h that rounds the other way is one of up to 128
    err = float((got - want).norm() / want.norm())
    del x, w13, w2, y, ws
    torch.cuda.empty_cache()
    assert err <= 1e-2, err


@pytest.mark.parametrize("rows", [1, 70, 200])
def test_training_forward_of_such_a_layer(rows):
    """The first projection of a training call, which keeps the factors of the backward pass as well, at every tile height."""
    import paper_2604_23108_amd as M
    T, d, F = rows, (1 << 24) + (1 << 20), 128
    if torch.cuda.mem_get_info()[0] < 60 << 30:
        pytest.skip("needs up to 50 GiB of free device memory")
    cfg = M.Config(T=T, d=d, n_groups=1, experts_per_group=1, d_ff=(F,), k_groups=1, k_experts=1,
                   select_mode=M.SELECT_PER_GROUP, dtype=M.BF16)
    gen = torch.Generator(device="cuda").manual_seed(9)
    normal = lambda *s: torch.randn(s, generator=gen, device="cuda").to(torch.bfloat16)
    idx = torch.cat([torch.arange(0, 32), torch.arange(d - 32, d)]).cuda()
    x, w13, w2 = (torch.zeros(s, dtype=torch.bfloat16, device="cuda") for s in ((T, d), (1, 2 * F, d), (1, d, F)))
    x[:, idx], w13[0, :, idx], w2[0, idx] = normal(T, len(idx)), normal(2 * F, len(idx)) * 0.1, normal(len(idx), F) * 0.1
    offsets = torch.tensor([0, T], dtype=torch.int32, device="cuda")
    y = torch.full((T, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    saved = torch.empty(M.mohge_workspace_size(cfg, M.CALL_FFN_SAVED), dtype=torch.uint8, device="cuda")
    print(f"[long rows, training] rows={rows}", flush=True)
    M.mohge_expert_ffn_train(cfg, x, None, offsets, [w13], [w2], y, saved)
    torch.cuda.synchronize()
    a, b = (x[:, idx].float() @ w13[0][:, idx].float().T.contiguous()).split(F, dim=1)
    want = (a * torch.sigmoid(a) * b).to(torch.bfloat16).float() @ w2[0][idx].float().T.contiguous()
    err = float((y[:, idx].float() - want).norm() / want.norm())
    zero = bool((y[:, 32:64] == 0).all())
    del x, w13, w2, y
    torch.cuda.empty_cache()
    assert err <= 1e-2 and zero, err      # (the bound of the test above)
