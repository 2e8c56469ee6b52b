"""Cloud building at the edges of its launch shapes (rows shorter and longer than a wave, one
voxel, the longest row, more levels than voxels) against the FP64 oracle, and clouds built in
the device memory of destroyed ones.

Tolerance: every level is three passes of positive terms, each with weights and products
rounded once and a compensated sum, so an element's relative error is at most a few units of
2^-24 per pass; 1e-6 holds that with room."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_1709_05418_amd as ds

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = ds.Context(0)
    yield c
    c.close()


def _density(dims, dtype, seed):
    g = torch.Generator().manual_seed(seed)
    d = (torch.rand((dims[2], dims[1], dims[0]), generator=g) - 0.2).clamp_min(0)
    d.view(-1)[0] = 0.75
    return d.to(dtype)


@pytest.mark.parametrize("dims,L,dtype", [
    ((1, 1, 1), 3, torch.float32), ((33, 20, 7), 8, torch.bfloat16),
    ((65, 3, 70), 4, torch.float32), ((5, 300, 4), 9, torch.bfloat16),
    ((4096, 2, 3), 13, torch.float32), ((64, 64, 130), 7, torch.float32)])
def test_levels_match_oracle_at_odd_sizes(ctx, dims, L, dtype):
    d = _density(dims, dtype, sum(dims))
    host = d.view(torch.int16).numpy().view(np.uint16) if dtype == torch.bfloat16 else d.numpy()
    amin, h0, sigma = (0.0, 0.0, 0.0), 0.01, 37.0
    grid = O.Grid(host, sigma, amin, h0)
    mean, _ = O.normalize(grid)
    pyr, pd, po = O.pyramid(grid, mean, L)
    c = ds.Cloud(ctx, d.cuda(), sigma, amin, h0, L, 3)
    try:
        assert c.info["mean_mu_t"] == pytest.approx(mean, rel=1e-6)
        assert ds.ds_cloud_majorant(c.h) == pytest.approx(sigma * float(d.float().max()), rel=1e-7)
        for i in range(L):
            ref = O.level(pyr, pd, po, i)
            got = c.level(i).cpu().numpy()
            assert got.shape == ref.shape
            assert np.all(np.abs(got - ref) <= 1e-6 * np.abs(ref) + 1e-30), i
    finally:
        c.close()


def test_reused_device_memory_changes_nothing(ctx):
    # a large cloud's memory, with its tracer and gather cells, goes to smaller and equal ones
    prm = ds.TracerParams(0.9, 0.5, 1.0)

    def everything(c, n):
        pos, view, light, _ = ds.ds_sample_records(c, cloud.h, n, 3)
        li, _ = ds.ds_trace_li(c, cloud.h, prm, pos, view, light, 8, 4)
        z, _ = ds.ds_gather(c, cloud.h, pos, view, light, 4)
        zp = ds.ds_gather_packed(c, cloud.h, pos, view, light, 4)
        return [t.cpu().numpy() for t in (pos, li, z, zp)]

    fresh = []
    for dims, seed in (((96, 90, 80), 1), ((96, 90, 78), 2), ((96, 90, 80), 3)):
        c = ds.Context(0)
        cloud = ds.Cloud(c, _density(dims, torch.float32, seed).cuda(), 50.0, (0., 0., 0.), 0.01, 5, 4)
        fresh.append(everything(c.h, 200))
        cloud.close()
        c.close()
    for _ in range(2):
        for k, (dims, seed) in enumerate((((96, 90, 80), 1), ((96, 90, 78), 2), ((96, 90, 80), 3))):
            cloud = ds.Cloud(ctx, _density(dims, torch.float32, seed).cuda(), 50.0, (0., 0., 0.), 0.01,
                             5, 4)
            for a, b in zip(everything(ctx.h, 200), fresh[k]):
                assert np.array_equal(a, b)
            cloud.close()
