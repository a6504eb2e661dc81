"""The decode form of the expert networks whose reduction is split over the waves of a workgroup: rows per
expert around its token blocks, reductions that leave waves without indices, column blocks cut short."""
import numpy as np
import pytest
import torch

import oracle
from synth import Workload, generate

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("counts", [(0, 1, 0, 0), (1, 0, 15, 16), (17, 0, 0, 15), (0, 0, 32, 0)])
@pytest.mark.parametrize("d,d_ff", [(64, (64, 128)), (192, (320, 64)), (1088, (192, 448)), (2112, (1600, 576))])
def test_skinny_split_edges(d, d_ff, counts):
    import paper_2604_23108_amd as M
    from gpu_harness import DeviceLayer
    T = sum(counts)
    w = Workload("split", T=T, d=d, n_groups=2, experts_per_group=2, d_ff=d_ff, k_groups=1, k_experts=1, seed=47)
    inp = generate(w)
    dl = DeviceLayer(w, inp, training=False, guard=True)
    L = dl.layer
    eidx = np.random.default_rng(5).permutation(np.repeat(np.arange(4), counts)).astype(np.int32).reshape(T, 1)
    M.mohge_permute(dl.cfg, torch.from_numpy(eidx).cuda(), L.counts, L.offsets, L.perm, L.inv_perm, None, None,
                    L.ws_permute)
    L.y_perm.fill_(float("nan"))
    print(f"[split] counts={counts} d={d} d_ff={d_ff}", flush=True)
    M.mohge_expert_ffn(dl.cfg, dl.x, L.perm, L.offsets, L.w13, L.w2, L.y_perm, L.ws_ffn)
    dl.check_guards()
    want = oracle.expert_ffn(w, inp.x.f32, [t.f32 for t in inp.w_gate], [t.f32 for t in inp.w_up],
                             [t.f32 for t in inp.w_down], np.arange(T, dtype=np.int32), eidx.reshape(-1))
    got, want = L.y_perm.float().cpu().numpy(), want[L.perm.cpu().numpy()]
    # h and y are rounded to bf16 once each: 2^-9 of the value and of a sum of such terms
    assert np.isfinite(got).all()
    assert np.abs(got - want).max() <= 8e-3 * np.abs(want).max()


@pytest.mark.parametrize("counts", [(0, 1, 0, 0), (1, 0, 15, 16), (17, 0, 0, 15)])
@pytest.mark.parametrize("d,d_ff", [(64, (64, 128)), (192, (320, 64)), (1088, (192, 448)), (2112, (1600, 576))])
def test_fp8_split_edges(d, d_ff, counts):
    """The same with FP8 weights (at these sizes the direct form), against the oracle on the dequantised weights."""
    import paper_2604_23108_amd as M
    from gpu_harness import DeviceLayer
    T = sum(counts)
    w = Workload("split8", T=T, d=d, n_groups=2, experts_per_group=2, d_ff=d_ff, k_groups=1, k_experts=1, seed=53)
    inp = generate(w)
    dl = DeviceLayer(w, inp, training=False, guard=True)
    L = dl.layer
    eidx = np.random.default_rng(5).permutation(np.repeat(np.arange(4), counts)).astype(np.int32).reshape(T, 1)
    M.mohge_permute(dl.cfg, torch.from_numpy(eidx).cuda(), L.counts, L.offsets, L.perm, L.inv_perm, None, None,
                    L.ws_permute)
    L.y_perm.fill_(float("nan"))
    L.use_fp8_weights()
    print(f"[fp8 split] counts={counts} d={d} d_ff={d_ff}", flush=True)
    M.mohge_expert_ffn_w8(dl.cfg, dl.x, L.perm, L.offsets, *L.w8, L.y_perm, L.ws_ffn)
    dl.check_guards()
    c13, s13, c2, s2 = ([t.cpu().numpy() for t in ts] for ts in L.w8)
    f32 = lambda v: np.ascontiguousarray(v, dtype=np.float32)
    w13 = [oracle.dequantize_rows(c, s) for c, s in zip(c13, s13)]
    want = oracle.expert_ffn(w, inp.x.f32, [f32(v[:, :F]) for v, F in zip(w13, d_ff)],
                             [f32(v[:, F:]) for v, F in zip(w13, d_ff)],
                             [f32(oracle.dequantize_rows(c, s)) for c, s in zip(c2, s2)],
                             np.arange(T, dtype=np.int32), eidx.reshape(-1))
    got, want = L.y_perm.float().cpu().numpy(), want[L.perm.cpu().numpy()]
    # the codes are exact in bf16; h and y are rounded to bf16 once each
    assert np.isfinite(got).all()
    assert np.abs(got - want).max() <= 8e-3 * np.abs(want).max()
