"""The path walker's launch shapes: a path's value does not depend on the team size, the
launch it falls in, or which other records are active, so a prefix of the records gives
bitwise the same estimates on its own (the oracle parity of the estimates themselves is in
test_gpu_tracer.py)."""
import numpy as np
import pytest

import paper_1709_05418_amd as ds
from paper_1709_05418_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def scene():
    import torch
    ctx = ds.Context(0)
    # extinction up to the box faces on one side, empty bricks on the other
    d = synth.cloud_density(40, 9)
    d[:, :, :20] = 0.5 + 0.5 * d[:, :, :20]
    amin, h0 = synth.unit_box(40)
    cloud = ds.Cloud(ctx, d.cuda(), 40.0, amin, h0, 4, 4)
    yield ctx, cloud
    torch.cuda.synchronize()
    cloud.close()
    ctx.close()


PRM = {"hg": ds.TracerParams(0.97, 0.85, 1.3), "direct": ds.TracerParams(0.9, 0.5, 0.7, 0, 0, 1),
       "env": ds.TracerParams(0.95, 0.3, 1.1, 1), "one": ds.TracerParams(0.95, 0.85, 1.0, 0, 1)}


# prefix and full sizes on both sides of 2^14 paths (teams of 16 and 8), whole and partial
# groups of 64 paths, and (the last) more paths than one launch takes (2^23)
@pytest.mark.parametrize("kind,few,many,spp", [
    ("hg", 1, 700, 33), ("hg", 100, 3000, 64), ("direct", 7, 300, 130), ("env", 65, 20000, 1),
    ("one", 128, 66000, 128)])
def test_prefix_of_records_is_bitwise_the_same(scene, kind, few, many, spp):
    ctx, cloud = scene
    pos, view, light, _ = ds.ds_sample_records(ctx.h, cloud.h, many, 5)
    p2, v2, l2, _ = ds.ds_sample_records(ctx.h, cloud.h, few, 5)
    for a, b in ((pos, p2), (view, v2), (light, l2)):
        assert np.array_equal(a[:few].cpu().numpy(), b.cpu().numpy())
    view[many // 2] = 0.0  # an unusable direction: estimate 0, others unchanged
    m1, s1 = ds.ds_trace_li(ctx.h, cloud.h, PRM[kind], pos, view, light, spp, 11)
    m2, s2 = ds.ds_trace_li(ctx.h, cloud.h, PRM[kind], p2, v2, l2, spp, 11)
    m1, s1 = m1.cpu().numpy(), s1.cpu().numpy()
    keep = np.arange(few) != many // 2
    assert np.array_equal(m1[:few][keep], m2.cpu().numpy()[keep])
    assert np.array_equal(s1[:few][keep], s2.cpu().numpy()[keep])
    assert m1[many // 2] == 0.0 and (m1 > 0).mean() > 0.5
    if kind == "one":  # records of the second launch, alone at the end of a shorter list
        n = 65600
        m3, _ = ds.ds_trace_li(ctx.h, cloud.h, PRM[kind], pos[:n], view[:n], light[:n], spp, 11)
        assert np.array_equal(m1[:n], m3.cpu().numpy())


def test_first_hits_do_not_depend_on_the_ray_count(scene):
    import torch
    ctx, cloud = scene
    g = torch.Generator().manual_seed(3)
    n = 40000
    d = torch.randn((n, 3), generator=g).cuda()
    o = (0.4 * torch.randn((n, 3), generator=g)).cuda()
    o = o - 2.0 * d / d.norm(dim=1, keepdim=True)
    d[17] = 0.0
    full = ds.ds_first_hits(ctx.h, cloud.h, PRM["hg"], (0.2, 0.9, 0.1), o, d, 3, 2)
    few = ds.ds_first_hits(ctx.h, cloud.h, PRM["hg"], (0.2, 0.9, 0.1), o[:100], d[:100], 3, 2)
    for a, b in zip(full, few):
        assert np.array_equal(a[:100].cpu().numpy(), b.cpu().numpy())
    hit = full[3].cpu().numpy()
    assert 0.1 < hit.mean() < 0.9 and hit[17] == 0 and not full[0][17].any()
