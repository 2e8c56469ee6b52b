"""Weight gradients of small networks over many rows, whose rows are split over workgroups: batches
at the edges of a split (128 rows), of the splits' number and of their last part, against the
oracles and within the bounds of test_gpu_chain.py; and a captured step of such a batch."""
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


# 6, 8 and 38 tiles: 106, 80 and 16 splits at most; 100 tiles (W = 200): 6
@pytest.mark.parametrize("K,W,H,B", [
    (1, 16, 1, 127), (1, 16, 1, 128), (1, 16, 1, 255), (1, 16, 1, 256), (1, 16, 1, 385),
    (1, 17, 2, 1023), (1, 64, 3, 4097), (1, 1, 1, 13569), (1, 16, 1, 13567), (6, 64, 3, 2047),
    (6, 33, 3, 2177), (2, 200, 2, 769), (2, 200, 2, 1021)])
def test_gradients_at_the_edges_of_splits(ctx, K, W, H, B):
    net, theta, z, t = _case(ctx, K, W, H, B)
    zt, tt = torch.from_numpy(z).cuda(), torch.from_numpy(t).cuda()
    args = theta, K, W, H, z.astype(np.float64), t.astype(np.float64)
    for prec, ref, tol in ((ds.DS_PREC_F32, O.loss_grad, 1e-5),
                           (ds.DS_PREC_BF16, _bf16_loss_grad, 1e-3)):
        lref, gref = ref(*args)
        ds.ds_net_set_train_precision(net.h, prec)
        loss, grad = ds.ds_loss_grad(net.h, zt, tt, net.n_params)
        e = rel_l2(grad.cpu().numpy(), gref)
        print(f"K={K} W={W} H={H} B={B} precision {prec}: grad rel_l2 {e:.2e}")
        assert loss.item() == pytest.approx(lref, rel=tol)
        assert e <= tol
    net.close()


def test_captured_step_of_a_split_batch():
    # eager steps of smaller batches between the replays leave the workspace where it is
    K, W, H, B = 1, 16, 1, 1000
    s = torch.cuda.Stream()
    ctx = ds.Context(0, stream=s)
    (net, _, z, t), (ref, _, _, _) = _case(ctx, K, W, H, B), _case(ctx, K, W, H, B)
    zt, tt = torch.from_numpy(z).cuda(), torch.from_numpy(t).cuda()
    loss = torch.zeros(1, device="cuda")
    torch.cuda.synchronize()
    opts = [ds.ds_adam_create(n.h) for n in (net, ref)]

    def same():
        torch.cuda.synchronize()
        assert np.array_equal(net.get_params(), ref.get_params())
    with torch.cuda.stream(s):
        for n, o in zip((net, ref), opts):
            ds.ds_net_set_train_precision(n.h, ds.DS_PREC_F32)
            ds.ds_train_step(n.h, o, zt, tt, loss)   # the workspace is either precision's
            ds.ds_net_set_train_precision(n.h, ds.DS_PREC_BF16)
        ds.ds_train_capture(net.h, opts[0], zt, tt, loss)
        for n in (900, 100, 1000):
            ds.ds_train_replay(opts[0])
            ds.ds_train_step(ref.h, opts[1], zt, tt, loss)
            same()
            for m, o in zip((net, ref), opts):
                ds.ds_train_step(m.h, o, zt[:n], tt[:n], loss)
            same()
    for o in opts:
        ds.ds_adam_destroy(o)
    for x in (net, ref, ctx):
        x.close()
