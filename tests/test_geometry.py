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
extern "C" void order(int gx, int G, int *cx, int *gy) {
    for (int l = 0; l < gx * G; ++l) chunk_order(l, gx, G, cx[l], gy[l]);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("geometry")
    (d / "geometry.cpp").write_text(SOURCE)
    so = d / "geometry.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, "-o", str(so),
                    str(d / "geometry.cpp")], check=True)
    return ctypes.CDLL(str(so))


@pytest.mark.parametrize("G", [8, 40, 1024])
def test_chunk_order(lib, G):
    """Every (chunk, row group) once; an XCD takes the row groups of a chunk in
    order, never comes back to a chunk, and touches the fewest chunks."""
    for gx in list(range(1, 41)) + [64, 100]:
        cx, gy = (np.empty(gx * G, np.int32) for _ in range(2))
        ptr = lambda a: a.ctypes.data_as(ctypes.POINTER(ctypes.c_int))  # noqa: E731
        lib.order(gx, G, ptr(cx), ptr(gy))
        assert np.array_equal(np.sort(cx * G + gy), np.arange(gx * G))
        for x in range(8):
            c, g = cx[x::8], gy[x::8]
            runs = np.flatnonzero(np.diff(c)) + 1
            assert len(np.unique(c)) == len(runs) + 1 <= -(-gx // 8) + 1
            for part in np.split(g, runs):
                assert np.array_equal(part, part[0] + np.arange(len(part)))
