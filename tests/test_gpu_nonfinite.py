"""A transmittance that has reached 0 does not stay 0 past an extinction that is not finite, or
whose ratio to the majorant overflows: ratio tracking multiplies on, 0 x infinity is no
number, and the estimate says so.  The cloud is thick enough that every transmittance through
it is 0 when it meets the bad layer, so a walk that stopped at 0 would give finite numbers."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_1709_05418_amd as ds

pytestmark = pytest.mark.gpu

# a majorant of 2^-6 and 16 mean free paths per voxel; -2e38 is 3.2e39 times the largest density
N, DENSITY, SIGMA, H0 = 16, 2.0 ** -4, 0.25, 1024.0


def _density(bad):
    d = torch.full((N, N, N), DENSITY)
    d[13:] = 0.0
    if bad is not None:
        d[12:14] = bad
    return d


@pytest.mark.parametrize("bad", [None, float("nan"), float("-inf"), -2e38])
def test_zero_transmittance_past_a_bad_layer(bad):
    ctx = ds.Context(0)
    d = _density(bad)
    cloud = ds.Cloud(ctx, d.cuda(), SIGMA, (0.0, 0.0, 0.0), H0, 1, 1)
    assert ds.ds_cloud_majorant(cloud.h) == SIGMA * DENSITY
    size = N * H0
    n = 200
    rng = np.random.default_rng(4)
    xy = (0.2 + 0.6 * rng.random((n, 2))) * size
    o = np.concatenate([xy, np.full((n, 1), -size)], 1).astype(np.float32)
    up = np.tile(np.float32([0, 0, 1]), (n, 1))
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    prm = ds.TracerParams(0.9, 0.5, 1.0)
    try:
        # camera rays from below collide near the bottom; the light shines through the layer
        for light, broken in (((0, 0, 1), bad is not None), ((0, 0, -1), False)):
            pos, _, direct, hit = ds.ds_first_hits(ctx.h, cloud.h, prm, light, t(o), t(up), 3)
            direct, hit = direct.cpu().numpy(), hit.cpu().numpy()
            assert hit.all() and (pos[:, 2].cpu().numpy() < 2 * H0).all()
            assert np.isnan(direct).all() if broken else np.isfinite(direct).all()
            # records: the same through every scattering's light sample
            rec = np.concatenate([xy, np.full((n, 1), 6 * H0)], 1).astype(np.float32)
            wl = np.tile(np.float32(light), (n, 1))
            got = []
            for few in (n, 20):   # teams of 8 and of 16
                m, _ = ds.ds_trace_li(ctx.h, cloud.h, prm, t(rec[:few]), t(up[:few]), t(wl[:few]),
                                      128, 7)
                m = m.cpu().numpy()
                assert np.isnan(m).all() if broken else np.isfinite(m).all()
                got.append(m)
            assert np.array_equal(got[0][:20], got[1], equal_nan=True)
            if bad != -2e38:      # the oracle's FP64 holds that ratio
                grid = O.Grid(d.numpy(), SIGMA, (0.0, 0.0, 0.0), H0)
                mo, _ = O.trace_li(grid, rec[:20], up[:20], wl[:20], albedo=0.9, g=0.5, spp=128,
                                   seed=7)
                assert np.array_equal(np.isnan(mo), np.isnan(got[1]))
    finally:
        cloud.close()
        ctx.close()
