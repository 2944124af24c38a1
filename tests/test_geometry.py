"""Launch geometry of the product kernels (csrc/geometry.h), compiled for the host."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1002_1202_amd", "csrc")

SOURCE = """
#include "geometry.h"
using namespace gsc;
extern "C" void order(int gx, int G, int ragged, int *cx, int *gy) {
    for (int l = 0; l < gx * G; ++l) chunk_order(l, gx, G, ragged, cx[l], gy[l]);
}
extern "C" int ragged(int end, int R, int width) { return ragged_end(end, R, width); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("geometry")
    (d / "geometry.cpp").write_text(SOURCE)
    so = d / "geometry.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, "-o", str(so),
                    str(d / "geometry.cpp")], check=True)
    return ctypes.CDLL(str(so))


def order(lib, gx, G, ragged):
    cx, gy = (np.empty(gx * G, np.int32) for _ in range(2))
    ptr = lambda a: a.ctypes.data_as(ctypes.POINTER(ctypes.c_int))  # noqa: E731
    lib.order(gx, G, ragged, ptr(cx), ptr(gy))
    return cx, gy


@pytest.mark.parametrize("ragged", [0, 1])
@pytest.mark.parametrize("G", [8, 40, 1024])
def test_chunk_order(lib, G, ragged):
    """Every (chunk, row group) once; an XCD takes the row groups of a chunk in
    order, never comes back to a full chunk, touches the fewest of them, and takes
    an eighth of a last chunk that is not full, spread over its sequence."""
    for gx in list(range(1, 41)) + [64, 100]:
        cx, gy = order(lib, gx, G, ragged)
        assert np.array_equal(np.sort(cx * G + gy), np.arange(gx * G))
        full = gx - ragged
        for x in range(8):
            c, g = cx[x::8], gy[x::8]
            if ragged:
                at, n = np.flatnonzero(c == full), np.arange(G // 8)
                assert np.array_equal(at, n + full * np.minimum(32 * (n // 32 + 1), G // 8))
                assert np.array_equal(g[c == full], x * G // 8 + n)
            c, g = c[c < full], g[c < full]
            runs = np.flatnonzero(np.diff(c)) + 1
            assert len(np.unique(c)) == (len(runs) + 1 if full else 0) <= -(-full // 8) + 1
            for part in np.split(g, runs) if full else []:
                assert np.array_equal(part, part[0] + np.arange(len(part)))


def test_ragged_end(lib):
    """A quarter of the last chunk empty, of 64 and of 128 columns."""
    assert [lib.ragged(192, R, 64) for R in (129, 176, 177, 192, 300)] == [1, 1, 0, 0, 0]
    assert [lib.ragged(256, R, 128) for R in (130, 224, 225, 256)] == [1, 1, 0, 0]
