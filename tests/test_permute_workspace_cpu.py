"""The permutation's workspace: one sized for a caller's largest batch serves all smaller ones (host code only)."""
import pytest

import paper_2604_23108_amd as M


@pytest.mark.parametrize("Ne", [1, 8, 24, 64, 256])
@pytest.mark.parametrize("k", [1, 4])
def test_workspace_never_falls_as_the_batch_grows(Ne, k):
    k = min(k, Ne)
    last = 0
    for T in sorted({int(1.09 ** i) + j for i in range(190) for j in (-1, 0, 1)} | set(range(0, 1100))):
        cfg = M.Config(T=T, d=64, n_groups=1, experts_per_group=Ne, d_ff=(64,), k_groups=1, k_experts=k,
                       select_mode=M.SELECT_GLOBAL, dtype=M.BF16)
        size = M.mohge_workspace_size(cfg, M.CALL_PERMUTE)
        assert size >= max(last, 4 * Ne * -(-T * k // 512)), T
        last = size
