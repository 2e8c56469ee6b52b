"""What the library does with device memory, on the CPU against a stand-in for the HIP runtime
(fake_hip.cpp): blocks of destroyed clouds, and calls that run out of memory.  Each test is
a child process with the stand-in loaded in front of the real runtime."""
import os
import subprocess
import sys
import textwrap

import pytest

import paper_1709_05418_amd as ds

HERE = os.path.dirname(os.path.abspath(__file__))
pytestmark = pytest.mark.skipif(not os.path.exists(ds.LIB_PATH),
                                reason="libdeepscatter.so not built")

PRELUDE = """
import ctypes as C, sys
sys.path.insert(0, {root!r})
F = C.CDLL({fake!r}, mode=C.RTLD_GLOBAL)
F.fake_live_bytes.restype = C.c_size_t
F.fake_limit.argtypes = F.fake_count.argtypes = [C.c_size_t]
import paper_1709_05418_amd as ds
L = ds.lib()
NONE = (1 << 64) - 1
MIB = 1 << 20
density = C.c_void_p(4096)   # never read: kernels do nothing here

def context():
    h = C.c_void_p()
    assert L.ds_create(0, None, C.byref(h)) == 0, ds.ds_last_error()
    return h

def cloud(ctx, n, K=2):
    h, amin = C.c_void_p(), (C.c_float * 3)(0, 0, 0)
    st = L.ds_cloud_create(ctx, density, 0, n, n, n, 1.0, amin, 1.0 / n, 2, None, K, C.byref(h))
    assert st == 0, ds.ds_last_error()
    return h

def free():
    return F.fake_live_bytes()
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("fake") / "libfakehip.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", os.path.join(HERE, "fake_hip.cpp"), "-o", out],
                   check=True)
    return out


@pytest.fixture
def run(fake):
    def go(body):
        code = PRELUDE.format(root=os.path.dirname(HERE), fake=fake) + textwrap.dedent(body)
        r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stdout + r.stderr
    return go


def test_the_next_cloud_takes_a_destroyed_ones_block(run):
    run("""
    ctx = context()
    F.fake_count(4 * MIB)
    a = cloud(ctx, 64); assert L.ds_cloud_destroy(a) == 0
    b = cloud(ctx, 64); assert F.fake_mallocs() == 1
    c = cloud(ctx, 64); assert F.fake_mallocs() == 2   # b holds the first block
    L.ds_cloud_destroy(b); L.ds_cloud_destroy(c); L.ds_destroy(ctx)
    assert F.fake_live_bytes() == 0
    """)


def test_a_block_that_could_not_be_waited_for_is_not_reused(run):
    # another stream may still read it
    run("""
    ctx = context()
    F.fake_count(4 * MIB)
    a = cloud(ctx, 64)
    F.fake_refuse(1, 0)
    assert L.ds_cloud_destroy(a) == 0
    F.fake_refuse(0, 0)
    assert F.fake_frees() == 1        # hipFree waits by itself
    b = cloud(ctx, 64)
    assert F.fake_mallocs() == 2
    L.ds_cloud_destroy(b)
    # a refused wait leaves no error for the next call
    assert L.ds_destroy(ctx) == 0 and F.fake_live_bytes() == 0
    """)


def test_a_block_that_could_be_neither_waited_for_nor_freed_is_set_aside(run):
    run("""
    ctx = context()
    F.fake_count(4 * MIB)
    a = cloud(ctx, 64)
    F.fake_refuse(1, 1)
    assert L.ds_cloud_destroy(a) == 0
    F.fake_refuse(0, 0)
    assert F.fake_frees() == 0
    b = cloud(ctx, 64)
    assert F.fake_mallocs() == 2      # not the first one's block
    L.ds_cloud_destroy(b); L.ds_destroy(ctx)
    assert F.fake_live_bytes() == 0   # and not lost
    """)


# What a call allocates: a network (parameters, packed copies), its fragments, Adam's moments,
# workspaces, a batch's order buffers, a light set, a phase table
CALLS = {
    "net": "lambda: L.ds_net_create(ctx, C.byref(ds._NetDesc(10, 200, 3)), C.byref(out))",
    "mlp": "lambda: L.ds_net_create_mlp(ctx, 10, 2, (C.c_int32 * 2)(200, 1), C.byref(out))",
    "params": "lambda: L.ds_net_set_params(net, theta, n)",
    "adam": "lambda: L.ds_adam_create(net, C.c_float(1e-3), C.c_float(.9), C.c_float(.999), C.c_float(1e-8), C.byref(out))",
    "gradient": "lambda: L.ds_loss_grad(net, density, density, 512, density, density)",
    "trace": "lambda: L.ds_trace_li(ctx, keep, C.byref(prm), density, density, density, C.c_int64(4096), 1024, C.c_uint64(1), density, None)",
    "predict": "lambda: L.ds_predict(ctx, keep, net, 0, density, density, density, C.c_int64(4096), density, None, None)",
    "lights": "lambda: L.ds_lights_create(ctx, 65536, dirs, irr, C.byref(out))",
    "cloud": "lambda: L.ds_cloud_create(ctx, density, 0, 64, 64, 64, C.c_float(1), (C.c_float * 3)(0, 0, 0), C.c_float(1 / 64), 2, None, 2, C.byref(out))",
    "context": "lambda: L.ds_create(0, None, C.byref(out))",
}


@pytest.mark.parametrize("owner", ["same", "other"])
@pytest.mark.parametrize("call", CALLS)
def test_kept_blocks_make_room_for_any_call(run, call, owner):
    # the memory that the call needs is held by a destroyed cloud's block alone
    run(f"""
    ctx = context()
    other = context()
    out = C.c_void_p()
    net = C.c_void_p()
    prm = ds.TracerParams(0.9, 0.85, 1.0)
    assert L.ds_net_create(ctx, C.byref(ds._NetDesc(2, 64, 3)), C.byref(net)) == 0
    n = ds.ds_net_param_count(2, 64, 3)
    theta = (C.c_float * n)()
    import numpy as np
    d3 = np.ones((65536, 3), np.float32); e1 = np.ones(65536)
    dirs, irr = C.c_void_p(d3.ctypes.data), C.c_void_p(e1.ctypes.data)
    keep = cloud(ctx, 8)
    owner = dict(same=ctx, other=other)[{owner!r}]
    a = cloud(owner, 150)
    L.ds_cloud_destroy(a)
    F.fake_limit(F.fake_live_bytes())
    F.fake_count(0)
    st = ({CALLS[call]})()
    assert st == 0, ds.ds_last_error()
    assert F.fake_mallocs() > 0 and F.fake_frees() > 0
    # the refused allocation leaves no error behind
    assert L.ds_synchronize(ctx) == 0 and F.hipGetLastError() == 0
    """)


def test_a_call_that_does_not_fit_still_says_so(run):
    run("""
    ctx = context()
    out = C.c_void_p()
    F.fake_limit(F.fake_live_bytes() + MIB)
    assert L.ds_net_create(ctx, C.byref(ds._NetDesc(10, 200, 3)), C.byref(out)) == -2
    assert "memory" in ds.ds_last_error()
    """)


def test_old_blocks_make_way_for_the_sizes_in_use(run):
    # once the list was full of blocks that fit no cloud, no new block entered it
    run("""
    ctx = context()
    start = F.fake_live_bytes()
    held = lambda: F.fake_live_bytes() - start
    for n in (200, 230, 260, 290, 320, 350, 380, 410, 440):   # no two within a quarter
        L.ds_cloud_destroy(cloud(ctx, n))
        assert held() <= (4 << 30) + MIB
    assert held() > 1 << 30
    F.fake_count(4 * MIB)
    L.ds_cloud_destroy(cloud(ctx, 470))      # 3.9 GB
    assert F.fake_mallocs() == 1 and held() <= (4 << 30) + MIB
    L.ds_cloud_destroy(cloud(ctx, 470))
    assert F.fake_mallocs() == 1             # the same block again
    # the oldest go first: a small block that was used last stays
    L.ds_cloud_destroy(cloud(ctx, 100))
    F.fake_count(4 * MIB)
    L.ds_cloud_destroy(cloud(ctx, 100))
    assert F.fake_mallocs() == 0
    # a block larger than the bound is not kept
    F.fake_count(1 << 32)
    L.ds_cloud_destroy(cloud(ctx, 700))
    assert F.fake_mallocs() == 1 and F.fake_frees() == 1
    L.ds_destroy(ctx)
    assert F.fake_live_bytes() <= start
    """)


def test_the_progressive_network_keeps_no_activations(run):
    # its layers are chained in one launch; the all-at-once MLPs keep three activations a row
    run("""
    ctx = context()
    net, mlp = C.c_void_p(), C.c_void_p()
    assert L.ds_net_create(ctx, C.byref(ds._NetDesc(2, 64, 3)), C.byref(net)) == 0
    assert L.ds_net_create_mlp(ctx, 2, 2, (C.c_int32 * 2)(64, 1), C.byref(mlp)) == 0
    rows = 65536
    at = free()
    assert L.ds_forward(ctx, net, density, C.c_int64(rows), density, density) == 0
    assert free() == at
    c = cloud(ctx, 8)
    assert L.ds_predict_reserve(ctx, c, net, 0, C.c_int64(64)) == 0   # the cloud's cells
    at = free()
    assert L.ds_predict_reserve(ctx, c, net, 0, C.c_int64(rows)) == 0
    held = free()
    assert abs(held - at - (rows - 64) * (4 * 451 + 1)) < 8192
    assert L.ds_predict(ctx, c, net, 0, density, density, density, C.c_int64(100000), density,
                        None, None) == 0
    assert free() == held
    assert L.ds_predict_reserve(ctx, c, mlp, 0, C.c_int64(rows)) == 0
    assert abs(free() - at - (rows - 64) * 4 * 451 - rows * 4 * 192) < 1 << 20
    """)
