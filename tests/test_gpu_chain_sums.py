"""BF16 gradients on both sides of the rule that forms a small batch's sums in two parts: 960 rows
at W = 200, 1344 at W = 130, 1808 at W <= 64, and 4032 for the scalar layer, against the
reference and within the bound of test_gpu_chain.py."""
import numpy as np
import pytest
import torch

import paper_1709_05418_amd as ds
from _util import rel_l2
from test_gpu_chain import _bf16_loss_grad, _case
from test_gpu_chain_widths import _biases

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,W,H,B", [(2, 200, 2, 960), (2, 200, 2, 961), (2, 130, 2, 1344),
                                     (2, 130, 2, 1345), (2, 64, 2, 1808), (2, 64, 2, 1809),
                                     (1, 130, 2, 4032), (1, 130, 2, 4033)])
def test_both_sides(K, W, H, B):
    ctx = ds.Context(0)
    net, theta, z, t = _case(ctx, K, W, H, B)
    ds.ds_net_set_train_precision(net.h, ds.DS_PREC_BF16)
    loss, grad = ds.ds_loss_grad(net.h, torch.from_numpy(z).cuda(), torch.from_numpy(t).cuda(),
                                 net.n_params)
    z, t = z.astype(np.float64), t.astype(np.float64)
    # (either side of ReLUs within 2e-5 of their corners: see test_gpu_chain_widths.py)
    refs = [_bf16_loss_grad(theta + s * _biases(K, W, H), K, W, H, z, t) for s in (0, 2e-5, -2e-5)]
    e = [rel_l2(grad.cpu().numpy(), g) for _, g in refs]
    print(f"K={K} W={W} H={H} B={B}: grad rel_l2", *(f"{x:.2e}" for x in e))
    assert loss.item() == pytest.approx(refs[0][0], rel=1e-3)
    assert min(e) <= 1e-3
    net.close()
    ctx.close()
