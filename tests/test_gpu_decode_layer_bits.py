"""The units of the single-launch decode layer walk the reduction alone, the separate launches split it over four
waves: the same bits, with one and two blocks of 16 rows per expert and reductions that leave quarters empty, uneven or
with a remainder."""
import numpy as np
import pytest
import torch

from synth import Workload, generate

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 16, 17, 32])
@pytest.mark.parametrize("d,d_ff", [(64, (64, 128)), (192, (320, 64)), (1088, (192, 448)), (2048, (576, 1024))])
def test_decode_layer_bits(d, d_ff, T):
    import paper_2604_23108_amd as M
    from gpu_harness import DeviceLayer
    w = Workload("dec_bits", T=T, d=d, n_groups=2, experts_per_group=3, d_ff=d_ff, k_groups=2, k_experts=2, seed=d + T)
    inp = generate(w)
    bias = np.zeros(w.n_experts, np.float32)
    bias[1] = 50.0                                          # every token of the first group on one expert
    inp.expert_logit_bias = bias
    dl = DeviceLayer(w, inp, training=False, guard=True)
    L, c = dl.layer, dl.layer.cfg
    print(f"[decode bits] T={T} d={d} d_ff={d_ff}", flush=True)
    y = L.forward_decode(dl.x).clone()
    torch.cuda.synchronize()
    assert M.mohge_fused_status(c, M.CALL_DECODE_LAYER, L.ws_decode) == 0, M.mohge_last_error()
    assert (L.expert_idx == 1).sum().item() == T
    L.y.fill_(float("nan"))
    M.mohge_permute(c, L.expert_idx, L.counts, L.offsets, L.perm, L.inv_perm, None, None, L.ws_permute)
    M.mohge_expert_ffn(c, dl.x, L.perm, L.offsets, L.w13, L.w2, L.y_perm, L.ws_ffn)
    M.mohge_combine(c, L.y_perm, L.inv_perm, L.gates, L.y)
    torch.cuda.synchronize()
    assert torch.isfinite(y.float()).all()
    assert torch.equal(y.view(torch.int16), L.y.view(torch.int16))
    dl.check_guards()
