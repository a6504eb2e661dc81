"""The router backward's reductions over tokens and its input gradient at the sizes where their splits
change: token counts around the splits and the waves of the weight gradients, rows from one to several
column blocks, more router rows than one pass of 32."""
import numpy as np
import pytest
import torch

import oracle
from synth import Workload, generate

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,n_groups,per_group", [(1, 64, 2, 2), (7, 192, 3, 5), (33, 320, 2, 16), (65, 2112, 4, 8),
                                                     (1030, 256, 8, 16), (2050, 1024, 2, 3)])
def test_route_backward_sizes(T, d, n_groups, per_group):
    import paper_2604_23108_amd as M
    from gpu_harness import DeviceLayer, from_dev, to_dev
    w = Workload("rbwd", T=T, d=d, n_groups=n_groups, experts_per_group=per_group, d_ff=(64,) * n_groups, k_groups=2,
                 k_experts=2, seed=T, training=True)
    inp = generate(w)
    dl = DeviceLayer(w, inp, backward=True, guard=True)
    L = dl.layer
    print(f"[route bwd] T={T} d={d}", flush=True)
    L.forward(dl.x)
    L.backward(dl.x, to_dev(inp.dy, True))
    torch.cuda.synchronize()
    dl.check_guards()
    # dW = dz^T x and dx = sum of the expert rows + dz W, from the device's own dz and rows
    dz = L.dz.double()
    x = dl.x.double()
    dw = torch.cat([L.dw_group, L.dw_expert]).double()
    want = dz.T @ x
    # fp32 sums of at most T terms: 2^-24 times the sum of the magnitudes, T / 32 terms in a chain
    bound = 2.0 ** -24 * (8 + T / 32) * (dz.abs().T @ x.abs())
    assert ((dw - want).abs() <= bound + 1e-30).all()
    wr = torch.cat([L.w_group, L.w_expert]).double()
    rows = L.dx_perm.double()[L.inv_perm.long()].reshape(T, w.k_experts, d).sum(1)
    want = rows + dz @ wr
    # one bf16 rounding (2^-9 relative) on top of fp32 sums
    assert ((L.dx.double() - want).abs() <= 2.0 ** -8 * want.abs() + 1e-5 * want.abs().max()).all()
