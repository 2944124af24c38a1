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
extern "C" void groups(int64_t nb, int chunks, int width, int64_t row_orbitals, int one_wave, int *out) {
    const RowGroups g = row_groups(nb, chunks, width, row_orbitals, one_wave);
    const int v[5] = {g.Gs, g.Gw, g.G1, g.G2, g.waves2};
    for (int i = 0; i < 5; ++i) out[i] = v[i];
}
extern "C" void asked(int64_t nb, int chunks, int groups, int *out) {
    RowGroups g = row_groups(nb, chunks, chunks, 68, false);
    set_groups(g, nb, groups);
    const int v[5] = {g.Gs, g.Gw, g.G1, g.G2, g.waves2};
    for (int i = 0; i < 5; ++i) out[i] = v[i];
}
extern "C" int small_full(int64_t N, int64_t K) { return small_full_carry(N, K); }
extern "C" int step(int64_t nb, int chunks, int64_t row_orbitals, int narrow) {
    return step_waves(nb, chunks, row_orbitals, narrow);
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


def groups(lib, nb, chunks, width, orbitals, one_wave):
    out = np.empty(5, np.int32)
    lib.groups(ctypes.c_int64(nb), chunks, width, ctypes.c_int64(orbitals), one_wave,
               out.ctypes.data_as(ctypes.POINTER(ctypes.c_int)))
    return out


@pytest.mark.parametrize("one_wave", [0, 1])
@pytest.mark.parametrize("chunks,width", [(1, 1), (2, 2), (4, 4), (8, 1), (24, 24)])
def test_row_groups(lib, chunks, width, one_wave):
    """Groups that leave partial sums hold at most four rows of one chunk (one a
    wave) however many rows there are, and one wave a row has no more groups than
    its rows fill, so that no XCD's share is empty."""
    for nb in [1, 3, 8, 9, 255, 256, 1023, 1024, 1025, 2048, 2049, 3072, 4096, 4097, 8192, 19038, 32768, 65536]:
        out = groups(lib, nb, chunks, width, 68, one_wave)
        Gs, Gw, G1, G2, waves2 = out
        slots = -(-nb // 4)
        assert (out[:4] % 8 == 0).all() and (out[:4] > 0).all()
        assert Gw == -(-min(nb, 65528) // 8) * 8
        if width * slots <= 16384:
            assert 4 * Gs >= nb and 4 * G1 >= nb and 4 * G2 >= nb
        assert G1 <= -(-slots // 8) * 8
        if waves2 == 1:
            assert G2 == G1
        if chunks * nb >= 4096 and not one_wave:
            assert Gs == G1             # four rows a group
        if one_wave:
            assert Gs == G1 and waves2 == 1


def test_step_waves(lib):
    """One wave a row for short rows in launches of one chunk with many rows."""
    step = lambda nb, chunks, orbitals, narrow: lib.step(ctypes.c_int64(nb), chunks, ctypes.c_int64(orbitals), narrow)  # noqa: E731
    assert [step(nb, 1, 68, 0) for nb in (4096, 12287, 12288, 32768)] == [4, 4, 1, 1]
    assert [step(nb, 1, 68, 1) for nb in (4095, 4096, 32768)] == [4, 1, 1]
    assert step(32768, 2, 68, 0) == step(32768, 2, 68, 1) == 4
    assert step(32768, 1, 162, 0) == step(32768, 1, 162, 1) == 4


def test_product_waves(lib):
    """The products with two matrices: one wave a row for short rows when there are
    enough of them; long rows are shared at every size."""
    waves = lambda nb, chunks, orbitals: groups(lib, nb, chunks, chunks, orbitals, 0)[4]  # noqa: E731
    assert [waves(nb, c, 68) for nb, c in ((4095, 1), (4096, 1), (2047, 2), (2048, 2), (32768, 8))] == [4, 1, 4, 1, 1]
    assert [waves(nb, c, 162) for nb, c in ((3000, 2), (3000, 3), (3000, 8), (12000, 1), (65536, 8))] == [4] * 5


def test_small_full_carry(lib):
    """Many shifts of the full carry go to the tiles."""
    fits = lambda N, K: lib.small_full(ctypes.c_int64(N), ctypes.c_int64(K))  # noqa: E731
    assert [fits(N, K) for N, K in ((512, 1280), (320, 2048), (4, 2048), (512, 64))] == [1] * 4
    assert [fits(N, K) for N, K in ((512, 1281), (321, 2048), (4, 2049), (384, 4096), (512, 65535))] == [0] * 5


def test_asked_row_groups(lib):
    """A caller's groups hold four rows in flight each, shared rows or not, and no
    group lies beyond the last row."""
    def asked(nb, g):
        out = np.empty(5, np.int32)
        lib.asked(ctypes.c_int64(nb), 2, g, out.ctypes.data_as(ctypes.POINTER(ctypes.c_int)))
        return out.tolist()
    assert asked(32768, 1024)[:4] == [1024, 4096, 1024, 1024]
    assert asked(4096, 1024)[:4] == [1024, 4096, 1024, 1024]
    assert asked(4096, 65528)[:4] == [1024, 4096, 1024, 1024]
    assert asked(19038, 8)[:4] == [8, 32, 8, 8]
    assert asked(72, 64)[:4] == [24, 72, 24, 24]
    assert asked(100000, 65528)[:4] == [25000, 65528, 25000, 25000]
    assert asked(1, 8)[:4] == [8, 8, 8, 8]
