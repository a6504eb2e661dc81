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
    # two fp32 dot products of at most 1024 terms, folded every 64: relative to the largest output the
    # rounding error stays below 2^-24 * (64 + 16) with room to spare
    assert np.isfinite(got).all()
    assert np.abs(got - want).max() <= 5e-6 * np.abs(want).max()
