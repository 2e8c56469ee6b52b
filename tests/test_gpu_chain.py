"""The layer chains at the edges of their tiles: widths around the 16-feature tiles (one wave
each), odd widths, one to three trailing layers, batches around the 16- and 32-row workgroups
and the rule between them (4096 rows), and the gradient's 64-row parts.  In FP32 outputs and
gradients against the FP64 oracle within the bound of the training parity tests, 1e-5 (sums of
some hundred terms through K + H layers).  With BF16 operands against the same operands summed
in FP64: what is left is FP32 sums, and about one value in 10^4 that lies so near the middle
of two BF16 numbers that it rounds the other way (2^-8 of itself, 4e-5 of a gradient's norm);
the bound is 1e-3."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_1709_05418_amd as ds
from paper_1709_05418_amd import synth
from _util import rel_l2

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = ds.Context(0)
    yield c
    c.close()


def _case(ctx, K, W, H, B):
    rng = np.random.default_rng(1000 * K + W + B)
    z = rng.random((B, 225 * K + 1)).astype(np.float32)
    theta = synth.init_params(K, W, H, K + W + H)
    _, pre = O.forward(theta.astype(np.float64), K, W, H, z)
    theta[-1] += np.float32(1.0 - np.percentile(pre, 30))  # most outputs past their ReLU
    net = ds.Net(ctx, K, W, H)
    net.set_params(theta)
    t = np.log1p(rng.random(B) * 1.5).astype(np.float32)
    return net, theta.astype(np.float64), z, t


def _bf16(x):
    return torch.from_numpy(x).to(torch.bfloat16).to(torch.float64).numpy()


def _pair(x, w):
    """x @ w.T with both operands as BF16 pairs, the product of the remainders left out."""
    xh, wh = _bf16(x), _bf16(w)
    return xh @ (wh + _bf16(w - wh)).T + _bf16(x - xh) @ wh.T


def _bf16_loss_grad(theta, K, W, H, z, t, nudge=0.0):
    """Loss and gradient with the operands of BF16 training, summed in FP64.  nudge: relative
    shift of the loss's derivative, which cancels in FP32."""
    p, at = {}, 0

    def take(name, *shape):
        nonlocal at
        n = int(np.prod(shape))
        p[name] = (slice(at, at + n), theta[at:at + n].reshape(shape))
        at += n
    for k in range(K):
        take(f"V{k}", W, 226)
        if k:
            take(f"W1{k}", W, W)
        for n in (f"b1{k}", f"W2{k}", f"b2{k}"):
            take(n, *((W, W) if n[0] == "W" else (W,)))
    for m in range(H):
        take(f"w{m}", 1 if m == H - 1 else W, W)
        take(f"b{m}", 1 if m == H - 1 else W)
    assert at == theta.size
    g, val = np.zeros_like(theta), {n: v for n, (_, v) in p.items()}

    def put(name, v):
        g[p[name][0]] = np.asarray(v).ravel()
    gamma, F, O_, x = z[:, -1:], [], [], np.zeros((len(z), W))
    zk = [np.concatenate([z[:, 225 * k:225 * (k + 1)], gamma], 1) for k in range(K)]
    for k in range(K):
        v = _bf16(zk[k][:, :225]) @ _bf16(val[f"V{k}"][:, :225]).T + gamma * val[f"V{k}"][:, 225]
        if k:
            v = v + _pair(x, val[f"W1{k}"])
        F.append(np.maximum(v + val[f"b1{k}"], 0))
        x = np.maximum(_pair(F[k], val[f"W2{k}"]) + val[f"b2{k}"] + x, 0)
        O_.append(x)
    Y = [x]
    for m in range(H - 1):
        Y.append(np.maximum(_pair(Y[m], val[f"w{m}"]) + val[f"b{m}"], 0))
    pre = _pair(Y[-1], val[f"w{H - 1}"]) + val[f"b{H - 1}"]
    out = np.maximum(pre, 0)
    r = np.log1p(out) - t[:, None]
    d = np.where(pre > 0, 2 * r / (len(z) * (1 + out)), 0) * (1 + nudge)
    for m in range(H - 1, -1, -1):
        put(f"w{m}", _bf16(d).T @ _bf16(Y[m]))
        put(f"b{m}", d.sum(0))
        d = _bf16(d) @ _bf16(val[f"w{m}"])
        if m:
            d = np.where(Y[m] > 0, d, 0)
    for k in range(K - 1, -1, -1):
        d = np.where(O_[k] > 0, d, 0)
        put(f"W2{k}", _bf16(d).T @ _bf16(F[k]))
        put(f"b2{k}", d.sum(0))
        dh = np.where(F[k] > 0, _bf16(d) @ _bf16(val[f"W2{k}"]), 0)
        put(f"V{k}", _bf16(dh).T @ _bf16(zk[k]))
        put(f"b1{k}", dh.sum(0))
        if k:
            put(f"W1{k}", _bf16(dh).T @ _bf16(O_[k - 1]))
            d = d + _bf16(dh) @ _bf16(val[f"W1{k}"])
    return float((r * r).mean()), g


@pytest.mark.parametrize("K,W,H,B", [
    (1, 1, 1, 1), (2, 1, 3, 5), (1, 15, 2, 15), (3, 16, 1, 16), (2, 17, 3, 17), (2, 33, 1, 33),
    (2, 64, 2, 64), (3, 129, 3, 65), (1, 200, 3, 31), (2, 256, 2, 500)])
def test_loss_and_gradients_at_tile_edges(ctx, K, W, H, B):
    net, theta, z, t = _case(ctx, K, W, H, B)
    zt, tt = torch.from_numpy(z).cuda(), torch.from_numpy(t).cuda()
    args = theta, K, W, H, z.astype(np.float64), t.astype(np.float64)
    for prec, ref, tol in ((ds.DS_PREC_F32, O.loss_grad, 1e-5),
                           (ds.DS_PREC_BF16, _bf16_loss_grad, 1e-3)):
        lref, gref = ref(*args)
        grefs = [gref]
        if prec == ds.DS_PREC_BF16:
            # every product takes the loss's derivative, rounded: in a small batch one row's
            # rounding the other way is up to 2^-8 of the norm, so either side is right
            grefs += [ref(*args, nudge)[1] for nudge in (2e-6, -2e-6)]
        ds.ds_net_set_train_precision(net.h, prec)
        loss, grad = ds.ds_loss_grad(net.h, zt, tt, net.n_params)
        e = min(rel_l2(grad.cpu().numpy(), g) for g in grefs)
        print(f"K={K} W={W} H={H} B={B} precision {prec}: loss {loss.item():.6f} ref {lref:.6f} "
              f"grad rel_l2 {e:.2e}")
        assert loss.item() == pytest.approx(lref, rel=tol)
        assert e <= tol
    net.close()


@pytest.mark.parametrize("K,W,H,P", [
    (1, 1, 1, 4097), (2, 17, 3, 4096), (2, 33, 2, 4111), (1, 256, 1, 4129), (3, 200, 3, 4113),
    (16, 256, 8, 4097)])  # the last: the most LDS
def test_forward_on_both_sides_of_the_row_rule(ctx, K, W, H, P):
    net, theta, z, _ = _case(ctx, K, W, H, P)
    zt = torch.from_numpy(z).cuda()
    out, pre = ds.ds_forward(ctx.h, net.h, zt)
    gref, pref = O.forward(theta, K, W, H, z.astype(np.float64))
    assert rel_l2(pre.cpu().numpy(), pref) <= 1e-5 and rel_l2(out.cpu().numpy(), gref) <= 1e-5
    # rows are independent and their sums ordered alike in either workgroup: bitwise the same
    few, fpre = ds.ds_forward(ctx.h, net.h, zt[-37:].contiguous())
    assert torch.equal(few, out[-37:]) and torch.equal(fpre, pre[-37:])
    net.close()
