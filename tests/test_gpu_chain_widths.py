"""The forward chain at the edges of its wave counts (up to 4 waves of 16 features, up to 12, from 13
on), which load the descriptors in groups of their own: many rows against the FP64 oracle within
the bound of test_gpu_chain.py and bitwise the last rows alone, and gradients in both precisions
against that file's references."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_1709_05418_amd as ds
from _util import rel_l2
from test_gpu_chain import _bf16_loss_grad, _case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = ds.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("K,W,H,P", [
    (1, 16, 1, 4110), (3, 48, 2, 4097), (2, 64, 3, 4129), (2, 65, 2, 4113), (2, 80, 1, 4111),
    (3, 160, 2, 4127), (2, 192, 3, 4097), (2, 193, 2, 4098)])
def test_forward_of_many_rows(ctx, K, W, H, P):
    net, theta, z, _ = _case(ctx, K, W, H, P)
    zt = torch.from_numpy(z).cuda()
    out, pre = ds.ds_forward(ctx.h, net.h, zt)
    gref, pref = O.forward(theta, K, W, H, z.astype(np.float64))
    assert rel_l2(pre.cpu().numpy(), pref) <= 1e-5 and rel_l2(out.cpu().numpy(), gref) <= 1e-5
    for n in (1, 17):
        few, fpre = ds.ds_forward(ctx.h, net.h, zt[-n:].contiguous())
        assert torch.equal(few, out[-n:]) and torch.equal(fpre, pre[-n:])
    net.close()


def _biases(K, W, H):
    """Which parameters of the canonical vector are hidden layers' biases."""
    m = []
    for k in range(K):
        m += [0] * (W * 226 + (W * W if k else 0)) + [1] * W + [0] * (W * W) + [1] * W
    for _ in range(H - 1):
        m += [0] * (W * W) + [1] * W
    return np.array(m + [0] * (W + 1), np.float64)


@pytest.mark.parametrize("K,W,H,B", [(2, 48, 2, 250), (2, 65, 2, 250), (2, 112, 2, 250),
                                     (2, 192, 2, 250), (2, 193, 2, 250)])
def test_gradients(ctx, K, W, H, B):
    net, theta, z, t = _case(ctx, K, W, H, B)
    zt, tt = torch.from_numpy(z).cuda(), torch.from_numpy(t).cuda()
    z, t = z.astype(np.float64), t.astype(np.float64)
    for prec, ref, tol in ((ds.DS_PREC_F32, O.loss_grad, 1e-5),
                           (ds.DS_PREC_BF16, _bf16_loss_grad, 1e-3)):
        lref, gref = ref(theta, K, W, H, z, t)
        grefs = [gref]
        if prec == ds.DS_PREC_BF16:
            # of some 2 10^5 ReLUs the nearest to its corner lies 10^-5 from it, no further than
            # the FP32 sum of 400 terms of size 1 (K + H layers deep) is from the FP64 one
            # (2, 193, 2: feature 81 of row 221), and one on its other side is 10^-3 of the
            # gradient: either side is right
            grefs += [ref(theta + s * _biases(K, W, H), K, W, H, z, t)[1] for s in (2e-5, -2e-5)]
        ds.ds_net_set_train_precision(net.h, prec)
        loss, grad = ds.ds_loss_grad(net.h, zt, tt, net.n_params)
        assert loss.item() == pytest.approx(lref, rel=tol)
        assert min(rel_l2(grad.cpu().numpy(), g) for g in grefs) <= tol
    net.close()
