"""The allocation-free FP32 prediction at the edges of its chunks: 3712 points of a ten-level
progressive network, 2880 of an all-at-once MLP of width 200, which keeps activations too.
Points are independent, so outputs, pre-activations and flags are bitwise ds_predict's."""
import pytest
import torch

import paper_1709_05418_amd as ds
from paper_1709_05418_amd import synth
from _util import Workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,chunk", [("progressive", 3712), ("mlp", 2880)])
def test_chunks(kind, chunk):
    w = Workload(32, 48.0, L=6, K=10, P=2 * chunk + 65, seed_cloud=9, seed_pts=90)
    ctx = ds.Context(0)
    cloud = ds.Cloud(ctx, w.density.cuda(), w.sigma_max, w.aabb_min, w.h0, w.L, w.K, w.mips)
    if kind == "mlp":
        net = ds.NetMLP(ctx, w.K, [200, 200, 1])
        net.set_params(0.02 * torch.randn(net.n_params, generator=torch.Generator().manual_seed(3)).numpy())
    else:
        net = ds.Net(ctx, w.K, 200, 3)
        net.set_params(synth.init_params(w.K, 200, 3, 17, branch_scale=0.3, out_scale=0.2,
                                         out_bias=0.5))
    pos, view, light = w.cuda_inputs()
    view[chunk] = 0.0  # an invalid point, the second chunk's first
    ds.ds_predict_reserve(ctx.h, cloud.h, net.h, ds.DS_PREC_F32, w.P)
    for n in (w.P, chunk, chunk + 1, 2 * chunk, 1):
        args = pos[:n], view[:n], light[:n]
        ref = ds.ds_predict(ctx.h, cloud.h, net.h, ds.DS_PREC_F32, *args)
        got = ds.ds_predict_f32_noalloc(ctx.h, cloud.h, net.h, *args)
        for a, b in zip(ref, got):
            assert torch.equal(a, b), (kind, n)
    for x in (net, cloud, ctx):
        x.close()
