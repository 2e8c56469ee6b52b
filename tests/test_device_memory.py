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
