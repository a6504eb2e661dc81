"""Where the router's bf16 matrix-core form starts: the forms that need no workspace ask for none (host code only)."""
import pytest

import paper_2604_23108_amd as M


def _workspace(T, d, n_groups, per_group, dtype=M.BF16):
    cfg = M.Config(T=T, d=d, n_groups=n_groups, experts_per_group=per_group, d_ff=(64,) * n_groups, k_groups=1, k_experts=1,
                   select_mode=M.SELECT_PER_GROUP, dtype=dtype)
    return M.mohge_workspace_size(cfg, M.CALL_ROUTE)


@pytest.mark.parametrize("n_groups,per_group,d,planes", [
    (2, 4, 128, False), (3, 4, 4096, False), (2, 7, 8192, False),            # one column tile of 16 router rows
    (3, 8, 128, False), (3, 8, 384, False), (3, 8, 512, True), (1, 31, 2048, True),
    (8, 4, 128, True), (4, 16, 4096, True),
    (4, 16, 1344, False),                                                    # not whole 128-deep chunks
])
def test_fp32_form_where_there_is_little_to_multiply(n_groups, per_group, d, planes):
    for T in (4097, 6000, 8191):
        assert (_workspace(T, d, n_groups, per_group) > 0) == planes, T
        assert _workspace(T, d, n_groups, per_group, M.F32) == 0
    assert _workspace(4096, d, n_groups, per_group) == 0
    # from 8192 tokens on always, and never less for more tokens
    rows = 4 * n_groups * (per_group + 1)
    sizes = [_workspace(T, d, n_groups, per_group) for T in (8192, 8193, 16384, 16385, 40000)]
    assert sizes == sorted(sizes)
    assert (sizes[0] >= 8192 * rows) == (d % 128 == 0)
