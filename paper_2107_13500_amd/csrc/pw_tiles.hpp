// Index arithmetic of the tiles: plain integers, the same on the host and in
// the kernels.  A plane holds up to 2^31 - 1 points, so every sum that could
// pass its last point is formed relative to a chunk's first one.
#pragma once

#include <stdint.h>

namespace pw {

// Points of one chunk of the march variant in the (j, k) run of a plane
// (column j = 0 first): `first` and how many follow, at most p.  A pair needs
// two points: with `pairs`, a last chunk of one starts a point early (never
// the only chunk, which has at least nz >= 2).
struct ChunkSpan {
    int32_t first, count;
};
__host__ __device__ inline ChunkSpan chunk_span(int32_t c, int32_t p, int32_t ny, int32_t nz, bool pairs) {
    const int32_t first = nz + c * p;                   // a point of the interior run: fits
    const int32_t left = (ny + 1) * nz - first;         // to the end of the interior run
    const int32_t early = pairs && left == 1 ? 1 : 0;
    return ChunkSpan{first - early, (left < p ? left : p) + early};
}

// 1-based level of the point `rel` points after `first` (which may lie up to
// one chunk past the last point of the plane).
__host__ __device__ inline int32_t point_level(int32_t first, int32_t rel, int32_t nz) {
    return (int32_t)(((uint32_t)first + (uint32_t)rel) % (uint32_t)nz) + 1;
}

// Split of nx planes into segments of at most `most` planes (any positive
// value): n = ceil(nx / most) segments of len = ceil(nx / n) planes, which
// start at or before plane nx and cover every plane (the last may be shorter).
struct SegmentSplit {
    int32_t n, len;
};
__host__ __device__ inline SegmentSplit segment_split(int32_t nx, int32_t most) {
    const uint32_t x = (uint32_t)nx, m = (uint32_t)(most < nx ? most : nx);
    const uint32_t n = (x + m - 1u) / m;
    return SegmentSplit{(int32_t)n, (int32_t)((x + n - 1u) / n)};
}

// Columns of the one-point x-y halo around nx x ny interior columns: up to
// 2^31 + 4 for the domains of a batch (nx ny < 2^30).
__host__ __device__ inline int64_t halo_columns(int32_t nx, int32_t ny) {
    return 2 * ((int64_t)nx + 2) + 2 * (int64_t)ny;
}

// Halo column h: first the rows j = 0 and j = ny + 1 over i = 0 .. nx + 1,
// then the planes i = 0 and i = nx + 1 over j = 1 .. ny.
struct Column {
    int32_t i, j;
};
__host__ __device__ inline Column halo_column(uint32_t h, int32_t nx, int32_t ny) {
    const uint32_t row = (uint32_t)nx + 2u, col = (uint32_t)ny;
    if (h < row) return Column{(int32_t)h, 0};
    if (h < 2u * row) return Column{(int32_t)(h - row), ny + 1};
    if (h < 2u * row + col) return Column{0, 1 + (int32_t)(h - 2u * row)};
    return Column{nx + 1, 1 + (int32_t)(h - 2u * row - col)};
}

}  // namespace pw
