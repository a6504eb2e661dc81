"""The backward of the gated combine with one to four slots per pass (small calls) and slot after slot (calls past
300 MB), against the definition."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("T,d", [(1, 64), (7, 1088), (330, 576), (131072, 448)])
def test_combine_backward_slots(T, d, k):
    import paper_2604_23108_amd as M
    cfg = M.Config(T=T, d=d, n_groups=1, experts_per_group=8, d_ff=(64,), k_groups=1, k_experts=k,
                   select_mode=M.SELECT_PER_GROUP, dtype=M.BF16)
    gen = torch.Generator(device="cuda").manual_seed(T + k)
    normal = lambda *s: torch.randn(s, generator=gen, device="cuda")
    dy, y_perm = normal(T, d).bfloat16(), normal(T * k, d).bfloat16()
    gates = torch.rand((T, k), generator=gen, device="cuda")
    inv = torch.randperm(T * k, generator=gen, device="cuda").int()
    dgates = torch.full((T, k), float("nan"), device="cuda")
    dy_perm = torch.full_like(y_perm, float("nan"))
    print(f"[combine bwd] T={T} d={d} K_e={k}", flush=True)
    M.mohge_combine_bwd(cfg, dy, y_perm, inv, gates, dgates, dy_perm)
    torch.cuda.synchronize()
    for s in range(k):
        rows = inv.view(T, k)[:, s].long()
        assert torch.equal(dy_perm[rows], (gates[:, s:s + 1] * dy.float()).bfloat16())      # one rounding of one product
        want = (dy.double() * y_perm[rows].double()).sum(1)
        # exact products of bf16 values; a lane adds at most 16 ceil(d / 512) of them, then six levels across the lanes
        bound = 2.0 ** -24 * (16 * -(-d // 512) + 6) * (dy.double() * y_perm[rows].double()).abs().sum(1)
        assert ((dgates[:, s].double() - want).abs() <= bound).all()
