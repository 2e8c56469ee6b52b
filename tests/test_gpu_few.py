"""The kernel for few points (up to 8192, four or sixteen to a workgroup) against the register
kernel, which a plan with a fixed grid always runs: outputs, pre-activations and flags bit by
bit, at every compiled width, on both sides of its two size rules, for points inside and
outside the box, unusable directions, an empty cloud and both point orders."""
import numpy as np
import pytest
import torch

import paper_1709_05418_amd as ds
from paper_1709_05418_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = ds.Context(0)
    yield c
    c.close()


def _points(P, amin, h0, n, seed):
    g = torch.Generator().manual_seed(seed)
    x = torch.tensor(amin) + n * h0 * (torch.rand(P, 3, generator=g) * 1.02 - 0.01)
    v, l = (torch.nn.functional.normalize(torch.randn(P, 3, generator=g)) for _ in range(2))
    if P > 2:
        x[P // 2, 0] = float("nan")
        v[P // 3] = 0.0
        l[P - 1] = v[P - 1]
    return [t.float().cuda().contiguous() for t in (x, v, l)]


@pytest.mark.parametrize("prec", ["bf16", "fp8"])
@pytest.mark.parametrize("K,W,H,counts", [
    (1, 1, 1, (1, 0)), (3, 16, 3, (4, 5)), (5, 32, 2, (17, 1006)), (6, 64, 3, (1000, 26)),
    (16, 100, 4, (37, 8155)), (10, 200, 3, (1025, 0)), (4, 256, 1, (333, 692)),
    (2, 250, 5, (8000, 192)), (2, 176, 3, (8193, 0)),
    (16, 256, 8, (1030, 7))])  # the last: the most LDS
def test_few_points_match_the_register_kernel(ctx, prec, K, W, H, counts):
    n = 24
    amin, h0 = synth.unit_box(n)
    clouds = [ds.Cloud(ctx, synth.cloud_density(n, 4 + i).cuda(), 24.0, amin, h0, K, K)
              for i in range(2)]
    net = ds.Net(ctx, K, W, H)
    net.set_params(synth.init_params(K, W, H, K + W))
    N = sum(counts)
    pts = _points(N, amin, h0, n, W)
    if prec == "fp8":
        ds.ds_net_quantize(ctx.h, net.h, clouds[0].h, ds.DS_PREC_FP8,
                           *_points(64, amin, h0, n, 1))
    prec = ds.DS_PREC_FP8 if prec == "fp8" else ds.DS_PREC_BF16
    b = ds.ds_batch_create(ctx.h, net.h, [c.h for c in clouds],
                           np.cumsum([0, *counts]).astype(np.int64))
    try:
        got = {}
        for order in (ds.DS_ORDER_INPUT, ds.DS_ORDER_SPATIAL):
            ds.ds_batch_set_order(b, order)
            for grid in (5, 0):
                ds.ds_batch_set_config(b, ds.DS_KERNEL_REGISTER, 4, grid)
                out, pre = (torch.full((N,), -1.0, device="cuda") for _ in range(2))
                flags = torch.full((N,), 77, dtype=torch.uint8, device="cuda")
                ds.ds_batch_predict(b, prec, *pts, out, pre, flags)
                got[order, grid] = out, pre, flags
        ref = got[ds.DS_ORDER_INPUT, 5]
        for key, arrays in got.items():
            for a, r in zip(arrays, ref):
                assert torch.equal(a, r), key
        if counts[1] == 0:  # the single-cloud call takes the same rule
            for a, r in zip(ds.ds_predict(ctx.h, clouds[0].h, net.h, prec, *pts), ref):
                assert torch.equal(a, r)
    finally:
        ds.ds_batch_destroy(b)
        net.close()
        for c in clouds:
            c.close()
