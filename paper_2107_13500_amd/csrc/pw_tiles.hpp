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
    const int64_t m = most < nx ? most : nx;
    const int64_t n = (nx + m - 1) / m;
    return SegmentSplit{(int32_t)n, (int32_t)((nx + n - 1) / n)};
}

}  // namespace pw
