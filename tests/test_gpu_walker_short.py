"""Short paths are walked one per thread, long ones by teams: the estimates are bitwise the same
either way.  A thin cloud lies between the rule's lines for few and for many paths, so a
prefix of a large call takes the other walk on its own; a thick one stays with teams."""
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


def _cloud(ctx, flights, n=40):
    """A cloud of `flights` mean free paths of its majorant across the box."""
    d = synth.cloud_density(n, 9)
    amin, h0 = synth.unit_box(n)
    return ds.Cloud(ctx, d.cuda(), flights / float(d.max()), amin, h0, 4, 4)


@pytest.fixture(scope="module")
def tables(ctx):
    _, p, _ = synth.cloud_droplet_phase(n_theta=901, n_r=40)
    full, chop = ds.Phase(ctx, p), ds.Phase(ctx, p, 5.0)
    rng = np.random.default_rng(8)
    dirs = rng.normal(size=(37, 3))
    lights = ds.Lights(ctx, dirs / np.linalg.norm(dirs, axis=1, keepdims=True),
                       rng.random(37) + 0.05)
    yield full, chop, lights
    for x in (full, chop, lights):
        x.close()


def _rays(n):
    g = torch.Generator().manual_seed(31)
    d = torch.randn((n, 3), generator=g)
    o = 0.3 * torch.randn((n, 3), generator=g) - 2.0 * d / d.norm(dim=1, keepdim=True)
    d[min(11, n - 1)] = 0.0  # an unusable ray
    return o.cuda(), d.cuda()


PRM = {"hg": (0.999, 0.85, 1.3), "direct": (0.97, 0.5, 0.7, 0, 0, 1), "env": (0.95, 0.3, 1.1, 1),
       "env direct": (0.95, 0.3, 1.1, 1, 0, 1), "cap": (0.95, 0.85, 1.0, 0, 2), "table": (0.97, 0.85, 1.0)}


# (environments and capped paths are short further up); spp below, at and past a partial sum
@pytest.mark.parametrize("kind,flights", [("hg", 10), ("direct", 10), ("env", 18),
                                          ("env direct", 18), ("cap", 14), ("table", 10)])
@pytest.mark.parametrize("spp", [1, 33, 130])
def test_records(ctx, tables, kind, flights, spp):
    cloud = _cloud(ctx, flights)
    few, many = 2000 // spp + 1, 700000 // spp
    prm = ds.TracerParams(*PRM[kind], **(dict(phase=tables[1]) if kind == "table" else {}))
    pos, view, light, _ = ds.ds_sample_records(ctx.h, cloud.h, many, 5)
    view[few // 2] = 0.0
    got = [[t.cpu().numpy()[:few] for t in ds.ds_trace_li(ctx.h, cloud.h, prm, pos[:n], view[:n],
                                                          light[:n], spp, 11)]
           for n in (many, few)]
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
    assert got[0][0][few // 2] == 0.0 and (got[0][0] > 0).any()
    cloud.close()


@pytest.mark.parametrize("table", [False, True])
@pytest.mark.parametrize("light", ["directional", "set", "environment"])
def test_pixels(ctx, tables, light, table):
    full, chop, lights = tables
    cloud = _cloud(ctx, 10 if light != "environment" else 18)
    o, d = _rays(20000)
    prm = ds.TracerParams(0.97, 0.85, 1.3, 1 if light == "environment" else 0,
                          **(dict(phase=chop, phase_first=full) if table else {}))
    got = []
    for n in (20000, 60):   # 660000 paths, 1980
        if light == "set":
            r = ds.ds_render_mc_lights(ctx.h, cloud.h, prm, lights.h, o[:n], d[:n], 33, 19)
        else:
            r = ds.ds_render_mc(ctx.h, cloud.h, prm, (0.2, 0.9, 0.1), o[:n], d[:n], 33, 19)
        got.append([t.cpu().numpy()[:60] for t in r])
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
    assert (got[0][0] > 0).mean() > 0.3 and got[0][0][11] == 0.0
    cloud.close()


@pytest.mark.parametrize("flights", [3, 40])
def test_first_hits(ctx, tables, flights):
    cloud = _cloud(ctx, flights)
    n = (1 << 18) + 77
    o, d = _rays(n)
    for prm in (ds.TracerParams(0.97, 0.85, 1.3),
                ds.TracerParams(0.97, 0.85, 1.3, phase=tables[1], phase_first=tables[0])):
        full = ds.ds_first_hits(ctx.h, cloud.h, prm, (0.2, 0.9, 0.1), o, d, 3, 2)
        few = ds.ds_first_hits(ctx.h, cloud.h, prm, (0.2, 0.9, 0.1), o[:900], d[:900], 3, 2)
        for a, b in zip(full, few):
            assert np.array_equal(a[:900].cpu().numpy(), b.cpu().numpy())
        hit = full[3].cpu().numpy()
        assert 0.05 < hit.mean() < 0.95 and hit[11] == 0
    cloud.close()


def test_record_draws(ctx):
    cloud = _cloud(ctx, 3)
    full = ds.ds_sample_records(ctx.h, cloud.h, 200000, 5)
    for n in (1, 500):
        for a, b in zip(full, ds.ds_sample_records(ctx.h, cloud.h, n, 5)):
            assert np.array_equal(a[:n].cpu().numpy(), b.cpu().numpy())
    assert (full[3].cpu().numpy() > 1).any()
    cloud.close()


def test_adaptive_rounds_change_walks(ctx):
    # many records in the first rounds, a few in the last: each result is the fixed count's
    cloud = _cloud(ctx, 10)
    pos, view, light, _ = ds.ds_sample_records(ctx.h, cloud.h, 3000, 5)
    prm = ds.TracerParams(0.97, 0.85, 1.3)
    m, v, n = ds.ds_trace_li_adaptive(ctx.h, cloud.h, prm, ds.Adaptive(64, 4096, 0.05, 1.96), pos,
                                      view, light, 11)
    n = n.cpu().numpy()
    assert n.min() < 1024 and n.max() == 4096
    for k in (int(n.min()), 4096):
        i = torch.from_numpy(np.flatnonzero(n == k)[:40]).cuda()
        j = int(i.max()) + 1     # a record's stream is its row
        mf, _ = ds.ds_trace_li(ctx.h, cloud.h, prm, pos[:j], view[:j], light[:j], k, 11)
        a, b = mf[i].cpu().numpy(), m[i].cpu().numpy()
        assert np.abs(a - b).max() <= 1e-12 * np.abs(b).max()
    cloud.close()
