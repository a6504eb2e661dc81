"""How many tokens the router backward adds in one fp32 chain, from the size of its workspace (host code only)."""
import pytest

import paper_2604_23108_amd as M


@pytest.mark.parametrize("T", [1, 33, 64, 777, 2048, 8192, 24576, 65536, 131072])
@pytest.mark.parametrize("d,n_groups,per_group", [(64, 1, 2), (1024, 8, 4), (1344, 5, 5), (2048, 3, 8), (4096, 4, 16),
                                                  (4096, 16, 16), (8192, 2, 32)])
def test_router_weight_gradient_chains(T, d, n_groups, per_group):
    cfg = M.Config(T=T, d=d, n_groups=n_groups, experts_per_group=per_group, d_ff=(64,) * n_groups, k_groups=1,
                   k_experts=1, select_mode=M.SELECT_PER_GROUP, dtype=M.BF16)
    Z = n_groups * (per_group + 1)
    up256 = lambda b: (b + 255) // 256 * 256
    ws = M.mohge_workspace_size(cfg, M.CALL_ROUTE_BWD)
    splits = (ws - up256(T * Z * 4)) // (Z * d * 4)
    assert splits >= 1
    # the measure: one chain per 64 tokens, at most 256 of them and at most 64 MB of partial sums, added by eight threads
    # in turn and then over the eight.  A chain of n additions costs n / 2 roundings of its sum.
    chains = max(1, min((T + 63) // 64, 256, (64 << 20) // (Z * d * 4)))
    measure = -(-T // chains) / 2 + chains / 16
    # here: four waves per split, each an even number of tokens; adding them costs (2 + 3 + 4) / 4
    per_wave = -(-(-(-T // splits)) // 8) * 2
    assert per_wave / 2 + 2.25 + splits / 16 <= max(measure, 8)
