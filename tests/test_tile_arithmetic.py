"""The kernels' tile arithmetic (csrc/pw_tiles.hpp) on the CPU, at the limits
of the shapes a plan accepts: compiled with the host compiler and compared
with Python integers."""
import ctypes
import os
import subprocess

import pytest

from paper_2107_13500_amd import build as hipbuild

WRAPPERS = """
#include "pw_tiles.hpp"
extern "C" {
void span(int32_t c, int32_t p, int32_t ny, int32_t nz, int32_t pairs, int32_t* out) {
    const pw::ChunkSpan s = pw::chunk_span(c, p, ny, nz, pairs != 0);
    out[0] = s.first;
    out[1] = s.count;
}
void split(int32_t nx, int32_t most, int32_t* out) {
    const pw::SegmentSplit s = pw::segment_split(nx, most);
    out[0] = s.n;
    out[1] = s.len;
}
int64_t halo(int32_t nx, int32_t ny) { return pw::halo_columns(nx, ny); }
void column(uint32_t h, int32_t nx, int32_t ny, int32_t* out) {
    const pw::Column c = pw::halo_column(h, nx, ny);
    out[0] = c.i;
    out[1] = c.j;
}
int32_t level(int32_t first, int32_t rel, int32_t nz) { return pw::point_level(first, rel, nz); }
}
"""


@pytest.fixture(scope="module")
def tiles(tmp_path_factory):
    d = tmp_path_factory.mktemp("tiles")
    src, lib = os.path.join(str(d), "tiles.cpp"), os.path.join(str(d), "tiles.so")
    with open(src, "w") as f:
        f.write(WRAPPERS)
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__host__=", "-D__device__=",
                    "-I", hipbuild.CSRC, src, "-o", lib], check=True)
    t = ctypes.CDLL(lib)
    t.halo.restype = ctypes.c_int64
    t.column.argtypes = [ctypes.c_uint32, ctypes.c_int32, ctypes.c_int32, ctypes.c_void_p]
    return t


def largest_ny(nz):
    """Rows of the largest plane a plan accepts: (ny + 2) nz < 2^31."""
    return (2 ** 31 - 1) // nz - 2


@pytest.mark.parametrize("chunk", [256, 512, 1024])
@pytest.mark.parametrize("nz", [2, 3, 64, 65, 96, 128, 255, 256])
def test_chunks_of_the_largest_planes_stay_inside_them(tiles, chunk, nz):
    out = (ctypes.c_int32 * 2)()
    for ny in (1, 7, 513, largest_ny(nz) - 1, largest_ny(nz)):
        points = ny * nz
        nchunks = -(-points // chunk)
        for c in {0, nchunks // 2, max(0, nchunks - 2), nchunks - 1}:
            for pairs in (0, 1):
                tiles.span(c, chunk, ny, nz, pairs, out)
                first, count = nz + c * chunk, min(chunk, points - c * chunk)
                if pairs and count == 1:
                    first, count = first - 1, 2
                assert tuple(out) == (first, count), (ny, c, pairs)
                assert first - nz >= 0 and first + count <= (ny + 1) * nz
                for rel in (0, count - 1, chunk - 1):   # lanes past the end of the chunk too
                    assert tiles.level(first, rel, nz) == (first + rel) % nz + 1


@pytest.mark.parametrize("most", [1, 2, 7, 16, 64, 2 ** 30, 2 ** 31 - 2, 2 ** 31 - 1])
def test_segments_cover_every_plane_for_any_bound(tiles, most):
    out = (ctypes.c_int32 * 2)()
    for nx in (1, 2, 3, 16, 17, 64, 1000, 2 ** 30 - 1, 2 ** 30):
        tiles.split(nx, most, out)
        n, length = out
        assert 1 <= length <= most and n >= 1
        assert (n - 1) * length < nx <= n * length, (nx, n, length)


def test_halo_columns_are_each_counted_once(tiles):
    out = (ctypes.c_int32 * 2)()
    for nx, ny in ((1, 1), (1, 5), (6, 1), (7, 4)):
        n = tiles.halo(nx, ny)
        seen = set()
        for h in range(n):
            tiles.column(h, nx, ny, out)
            seen.add(tuple(out))
        want = {(i, j) for i in range(nx + 2) for j in range(ny + 2) if i in (0, nx + 1) or j in (0, ny + 1)}
        assert seen == want and n == len(want)


@pytest.mark.parametrize("nx,ny", [(2 ** 30 - 1, 1), (1, 2 ** 30 - 1), (2 ** 29, 2)])
def test_halo_columns_of_the_longest_domains(tiles, nx, ny):
    """Domains of nearly 2^31 points two levels deep: the count passes 2^31."""
    out = (ctypes.c_int32 * 2)()
    n = tiles.halo(nx, ny)
    assert n == 2 * (nx + 2) + 2 * ny
    for h, want in ((nx + 1, (nx + 1, 0)), (2 * nx + 3, (nx + 1, ny + 1)), (n - 1, (nx + 1, ny)),
                    (n - 1 - ny, (0, ny))):
        tiles.column(h, nx, ny, out)
        assert tuple(out) == want
