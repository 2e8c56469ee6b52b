"""The path tracer's random words by position against the oracle's serial stream, on the CPU
(stream.h compiled as host code): around the start, where the first counter word of the
blocks carries (2^34 words), and where 32 bits of word position end (2^32 words)."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

import oracle as O
import paper_1709_05418_amd as ds

CSRC = os.path.join(os.path.dirname(ds.__file__), "csrc")
CODE = """
#include "stream.h"
using namespace ds;
// n words from position q on, as the walker reads them: a window of four lanes at a time
template <int KIND> static void read(uint64_t seed, uint64_t id, uint64_t at, int n, uint32_t *out)
{
    WordPos<KIND> q = (WordPos<KIND>)at;
    while (n > 0) {
        int x = (int)(q & 3);
        for (uint32_t i = 0; i < 4; ++i) {
            uint32_t b[4];
            stream_block(seed, (uint32_t)id, (uint32_t)(id >> 32), (q >> 2) + i, b);
            for (int c = 0; c < 4; ++c)
                if (4 * (int)i + c >= x && n > 0)
                    *out++ = b[c], --n;
        }
        q = (q & ~(WordPos<KIND>)3) + 16;
    }
}
extern "C" void record_draw(uint64_t seed, uint64_t id, uint64_t at, int n, uint32_t *out)
{
    read<kRecordDraws>(seed, id, at, n, out);
}
extern "C" void record_path(uint64_t seed, uint64_t id, uint64_t at, int n, uint32_t *out)
{
    read<kRecordPaths>(seed, id, at, n, out);
}
"""


@pytest.fixture(scope="module")
def words(tmp_path_factory):
    d = tmp_path_factory.mktemp("stream")
    (d / "w.cpp").write_text(CODE)
    out = str(d / "libw.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__host__=", "-D__device__=",
                    "-D__forceinline__=inline", "-I", CSRC, str(d / "w.cpp"), "-o", out], check=True)
    return C.CDLL(out)


@pytest.mark.parametrize("kind,at", [
    ("record_draw", 0), ("record_draw", 3), ("record_draw", (1 << 32) - 21),
    ("record_draw", (1 << 34) - 18), ("record_draw", (1 << 40) + 5), ("record_path", 0),
    ("record_path", (1 << 30) - 7)])
def test_words_follow_the_stream(words, kind, at):
    seed, rec, n = 0x123456789ABCDEF1, (77 << 20) + 5, 40
    got = np.zeros(n, np.uint32)
    getattr(words, kind)(C.c_uint64(seed), C.c_uint64(rec), C.c_uint64(at), n,
                         got.ctypes.data_as(C.c_void_p))
    key = np.array([seed & 0xFFFFFFFF, seed >> 32], np.uint32)
    ref = []
    for b in range(at // 4, (at + n) // 4 + 1):
        ref += list(O.philox(np.array([rec, 0, b & 0xFFFFFFFF, b >> 32], np.uint32), key))
    assert np.array_equal(got, np.array(ref[at % 4:at % 4 + n], np.uint32))
