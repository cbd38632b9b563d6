// Batched PW advection: many uneven subdomains in one launch, plus the
// periodic halo fill and the field perturbation used between repeated
// timestep calls.
//
// The plan flattens every domain's (chunk, segment) tiles into one global
// tile range (prefix sums in a device table).  By default one workgroup runs
// each tile (longest tiles first, handed to the XCDs in runs of neighbouring
// tiles); on request a persistent grid sized to the GPU walks the range
// instead (each XCD a contiguous share).  Each workgroup maps a tile to its
// domain (a binary search, then a forward scan) and runs the per-tile code
// of the single-domain march kernel.  The per-point arithmetic
// is the same source, and the library is built with FMA formed only within
// a source expression, so each domain's result is bit-identical to a
// pw_advect call (the result of a point does not depend on the tiling).
//
// Each domain splits its x range into segments of even length (at most the
// plan's segment length) rather than full segments and a short last one:
// tiles of equal length keep the workgroups that run neighbouring chunks in
// step, so the y-halo columns and boundary planes they share are still in L2
// when the second one reads them (measured on the 384-domain batch: 3-6%
// faster for FP64, FP32 and BF16).
//
// The tile list takes the domains longest tiles first (by segment length,
// then in the caller's order; each domain's tiles stay together), so the
// short tiles fill the end of the launch instead of a few long ones running
// alone.  The table row of a domain keeps the index of its record.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <mutex>
#include <vector>

#include "pw_plan.hpp"

namespace pw {

__host__ __device__ inline void domain_tiles(int32_t nx, int32_t ny, int32_t nz, int32_t chunk, int32_t seg_max,
                                             BatchDomain* b);

namespace {

__device__ __forceinline__ bool shape_matches(const pw_shape& a, const BatchDomain& b) {
    const int64_t sy = a.sy ? a.sy : a.nz;
    const int64_t sx = a.sx ? a.sx : (int64_t)(a.ny + 2) * sy;
    return a.nx == b.nx && a.ny == b.ny && a.nz == b.nz && a.reserved == 0 && sy == b.sy && sx == b.sx;
}

__device__ __forceinline__ float scale_or_one(float s) { return s > 0.0f ? s : 1.0f; }

// A record's scale must be 0 (meaning 1) or a finite positive power of two
// (normal or subnormal), as pw_advect requires of its scales; folding such
// scales into the coefficients is exact.
__device__ __forceinline__ bool scale_ok(float s) {
    const uint32_t b = __float_as_uint(s);
    if (b == 0u) return true;                       // +0: default scale
    if (b >> 31) return false;                      // negative or -0
    const uint32_t e = (b >> 23) & 0xffu, m = b & 0x7fffffu;
    if (e == 0xffu) return false;                   // Inf or NaN
    return e != 0u ? m == 0u : __popc(m) == 1;
}

__device__ __forceinline__ bool scales_ok(const pw_scales& sc) {
    bool ok = true;
#pragma unroll
    for (int f = 0; f < 3; ++f) ok = ok && scale_ok(sc.in_scale[f]) && scale_ok(sc.out_scale[f]);
    return ok;
}

template <typename ST>
__device__ __forceinline__ DomainArgs domain_from(const pw_domain_args& a, const BatchDomain& b) {
    DomainArgs d{};
    d.u = a.u;
    d.v = a.v;
    d.w = a.w;
    d.su = a.su;
    d.sv = a.sv;
    d.sw = a.sw;
    d.tzc1 = a.tzc1;
    d.tzc2 = a.tzc2;
    d.tzd1 = a.tzd1;
    d.tzd2 = a.tzd2;
    float in_s[3], out_s[3];
    for (int f = 0; f < 3; ++f) {
        in_s[f] = scaled_type<ST>::value ? scale_or_one(a.scales.in_scale[f]) : 1.0f;
        out_s[f] = scaled_type<ST>::value ? scale_or_one(a.scales.out_scale[f]) : 1.0f;
    }
    fold_coefficients(a.tcx, a.tcy, in_s, out_s, d.cx, d.cy, d.cz);
    d.nx = b.nx;
    d.ny = b.ny;
    d.nz = b.nz;
    d.sy = b.sy;
    d.sx = b.sx;
    return d;
}

// The last row whose `begin` (its first tile or workgroup) is at most t.
template <typename T>
__device__ __forceinline__ int find_domain(const BatchDomain* table, int ndom, T t, T BatchDomain::*begin) {
    int lo = 0, hi = ndom - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (table[mid].*begin <= t) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

__device__ __forceinline__ bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Which per-tile code paths a batched kernel carries.  Every path inlined
// into the batched kernel counts towards its register allocation, so a
// plan launches the kind its shapes need:
//   kFixedNz  column heights 64 / 96 / 128 only, every vector aligned;
//   kEven0..  even heights of at most kHeightClass[kind - kEven0] and any
//             element alignment: the one run-time-height path of the class of
//             the tallest column;
//   kClass0.. likewise for any heights.
// If every shape allows aligned vectors (vec_shapes), every field pointer must
// be 16-byte aligned; a record that is not is skipped and counted like a
// shape mismatch.
enum BatchKind { kFixedNz = 0, kEven0 = 1, kEven1 = 2, kEven2 = 3, kClass0 = 4, kClass1 = 5, kClass2 = 6 };
constexpr int kind_class(int kind) { return kind >= kClass0 ? kind - kClass0 : kind - kEven0; }

// gate: NULL, or a device word that must be nonzero for the launch to run
// (the allocation-free entry point's table check); if it is zero, workgroup
// 0 counts every domain as skipped and all workgroups exit.
// Tile order of one workgroup per tile (kOneTileRuns): XCD x of block g of
// the tile list takes tiles g 8R + x R .. g 8R + x R + R - 1, one per
// workgroup in dispatch order, so all XCDs work in the same window of the
// list at a time while runs of R neighbouring chunks meet in one XCD's L2;
// the grid is padded to whole blocks and workgroups past the last tile exit.
// Measured on the 384-domain batch against plain dispatch order: as fast or
// up to 1% faster, and the y-halo re-reads of neighbouring chunks hit L2.
constexpr int kOneTileRuns = 8;

// wg_per_cu 0 (the default) or PW_WG_ONE_PER_TILE: one workgroup per tile;
// 1..8: a persistent grid of that many workgroups per CU.
inline bool batched_one_per_tile(const pw_tuning& t) { return t.wg_per_cu <= 0; }

template <typename ST, int NT, int P, int KIND>
__global__ __launch_bounds__(NT) void pw_batched_kernel(const BatchDomain* __restrict__ table, int ndom,
                                                        int64_t ntiles, const pw_domain_args* __restrict__ args,
                                                        unsigned long long* errors,
                                                        int vec_shapes, int one_per_tile, const int32_t* __restrict__ order,
                                                        const uint32_t* gate, unsigned long long* bump) {
    using CT = typename compute_of<ST>::type;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    CT* lds = reinterpret_cast<CT*>(smem_raw);
    if (bump != nullptr && blockIdx.x == 0 && threadIdx.x == 0) *bump += 1ull;   // a timestep's call counter
    if (gate != nullptr && *gate == 0u) {   // uniform over the grid
        if (blockIdx.x == 0 && threadIdx.x == 0) atomicAdd(errors, (unsigned long long)ndom);
        return;
    }
    // Persistent grid: workgroups are dispatched round-robin over the XCDs;
    // each XCD gets a contiguous share of the tile range, walked by its own
    // workgroups, so the tiles in flight on one XCD are neighbouring chunks
    // and segments of the same domains and share their halo columns and
    // planes in its L2.
    const int G = (int)gridDim.x;
    const int x = (int)blockIdx.x % kNumXcd;
    const int slot = (int)blockIdx.x / kNumXcd;
    const int q = G / kNumXcd, r = G % kNumXcd;
    const int wgs = q + (x < r ? 1 : 0);                 // workgroups on this XCD
    const int before = x * q + (x < r ? x : r);          // workgroups on lower XCDs
    int64_t t_begin = ntiles * before / G + slot, t_end = ntiles * (before + wgs) / G, t_step = wgs;
    if (one_per_tile) {
        int64_t t;
        if (order != nullptr) {
            t = order[blockIdx.x];   // the plan's dispatch order; -1: no tile
        } else {
            const int64_t sl = blockIdx.x / kNumXcd;
            t = (sl / kOneTileRuns) * (kNumXcd * kOneTileRuns) + (int64_t)x * kOneTileRuns + sl % kOneTileRuns;
        }
        t_begin = t < 0 ? 0 : t;
        t_end = (t >= 0 && t < ntiles) ? t + 1 : t_begin;   // no tile: empty range
        t_step = 1;
    }
    int dom = -1;
    for (int64_t t = t_begin; t < t_end; t += t_step) {
        // tiles only move forward: after the first binary search a short
        // forward scan finds the domain (usually zero or one step)
        if (dom < 0) {
            dom = find_domain(table, ndom, t, &BatchDomain::tile_begin);
        } else {
            while (dom + 1 < ndom && table[dom + 1].tile_begin <= t) ++dom;
        }
        const BatchDomain b = table[dom];
        const int64_t local = t - b.tile_begin;
        const int c = (int)(local % b.nchunks);
        const int s = (int)(local / b.nchunks);
        const pw_domain_args& a = args[b.rec];
        if (!shape_matches(a.shape, b) || !a.u || !a.v || !a.w || !a.su || !a.sv || !a.sw ||
            (scaled_type<ST>::value && !scales_ok(a.scales))) {
            if (threadIdx.x == 0 && local == 0) atomicAdd(errors, 1ull);
            continue;   // uniform over the workgroup
        }
        const DomainArgs d = domain_from<ST>(a, b);
        const int i_begin = 1 + s * b.seg;   // <= nx: (nseg - 1) * seg < nx
        const int i_end = min(i_begin + b.seg - 1, b.nx);
        const bool vec = aligned16(a.u) && aligned16(a.v) && aligned16(a.w) && aligned16(a.su) &&
                         aligned16(a.sv) && aligned16(a.sw);
        if (vec_shapes && !vec) {
            if (threadIdx.x == 0 && local == 0) atomicAdd(errors, 1ull);
            continue;   // uniform over the workgroup
        }
        // Short tiles leave less time to hide a plane's latency: FP64
        // compute (three LDS slots) keeps three planes in flight, and every
        // storage type takes the branch-free data movement, whose exact
        // outstanding-load counts keep those planes in flight (measured on
        // the 384-domain batch: FP64 1.45 -> 1.22 ms, FP32 0.75 -> 0.64 ms).
        constexpr int D = march_slots<CT>() == 3 ? 3 : 2;
        constexpr bool X = true;
        if constexpr (KIND != kFixedNz) {
            march_tile<ST, NT, P, -kHeightClass[kind_class(KIND)], (KIND < kClass0), D, X>(d, c, i_begin, i_end, lds);
        } else if (b.nz == 64) {
            march_tile<ST, NT, P, 64, true, D, X>(d, c, i_begin, i_end, lds);
        } else if (b.nz == 96) {
            march_tile<ST, NT, P, 96, true, D, X>(d, c, i_begin, i_end, lds);
        } else {
            march_tile<ST, NT, P, 128, true, D, X>(d, c, i_begin, i_end, lds);
        }
    }
}

// Storage elements moved as raw bits through global pointers (the storage
// structs cannot be assigned through an address-space-qualified lvalue).
template <int N> struct bits_of;
template <> struct bits_of<2> { using type = uint16_t; };
template <> struct bits_of<4> { using type = uint32_t; };
template <> struct bits_of<8> { using type = uint64_t; };
template <typename ST> using storage_bits = typename bits_of<sizeof(ST)>::type;
template <typename ST> __device__ __forceinline__ ST from_bits(storage_bits<ST> u) {
    ST x;
    __builtin_memcpy(&x, &u, sizeof(ST));
    return x;
}
template <typename ST> __device__ __forceinline__ storage_bits<ST> to_bits(ST x) {
    storage_bits<ST> u;
    __builtin_memcpy(&u, &x, sizeof(ST));
    return u;
}

// Periodic x-y halo of u, v, w.  Each halo column (i, j) copies interior
// column (wrap(i), wrap(j)) with wrap(0) = n, wrap(n + 1) = 1 -- the same
// result as filling x faces first and then y faces over the halo'd x range.
// grid: y over domains, x a number of workgroups sized to the mean domain's
// halo; each workgroup strides over its domain's halo elements (every
// element is written once, from an interior source, so the order is free).
template <typename ST>
__global__ __launch_bounds__(256) void pw_halo_kernel(const BatchDomain* __restrict__ table,
                                                      const pw_domain_args* __restrict__ args) {
    const BatchDomain b = table[blockIdx.y];
    const pw_domain_args& a = args[b.rec];
    if (!shape_matches(a.shape, b) || !a.u || !a.v || !a.w) return;
    using U = storage_bits<ST>;
    global_ptr<U> f[3] = {as_global((U*)a.u), as_global((U*)a.v), as_global((U*)a.w)};
    const int64_t n = halo_columns(b.nx, b.ny) * b.nz;
    for (int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x; g < n; g += (int64_t)gridDim.x * 256) {
        const int k = (int)(g % b.nz);
        const Column at = halo_column((uint32_t)(g / b.nz), b.nx, b.ny);
        const int i = at.i, j = at.j;
        const int si = i == 0 ? b.nx : (i == b.nx + 1 ? 1 : i);
        const int sj = j == 0 ? b.ny : (j == b.ny + 1 ? 1 : j);
        const int64_t dst = k + (int64_t)j * b.sy + (int64_t)i * b.sx;
        const int64_t src = k + (int64_t)sj * b.sy + (int64_t)si * b.sx;
#pragma unroll
        for (int q = 0; q < 3; ++q) f[q][dst] = f[q][src];
    }
}

// SplitMix64 finaliser (Steele, Lea and Flood, OOPSLA 2014).
__host__ __device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
    x += 0x9e3779b97f4a7c15ull;
    x = (x ^ (x >> 30)) * 0xbf58476d1ce4e5b9ull;
    x = (x ^ (x >> 27)) * 0x94d049bb133111ebull;
    return x ^ (x >> 31);
}

// 32-bit integer hash "lowbias32" (C. Wellons, "Prospecting for Hash
// Functions", 2018).
__device__ __forceinline__ uint32_t lowbias32(uint32_t x) {
    x ^= x >> 16;
    x *= 0x7feb352du;
    x ^= x >> 15;
    x *= 0x846ca68bu;
    x ^= x >> 16;
    return x;
}

// u += amp * r, v += amp * r' on the interior, r uniform in [-1, 1) from a
// counter-based hash of (seed, call, domain, field, point); `call` is read
// from device memory so a captured graph perturbs differently on each replay.
// The (seed, call, domain) key is mixed once by SplitMix64; each element then
// costs one 32-bit hash of its field and its point index g = k + nz ((j - 1) +
// ny (i - 1)), so the values do not depend on how the work is split.
// One workgroup per chunk of the (j, k) points of a plane times at most
// `planes` x planes, a split of its own (find_domain by fill_begin): the
// advection's tiles may be long, and their number too small to fill the chip.
// Each thread reads the points of kPerturbPlanes planes before it writes them.
//
// HALO (the recorded timestep): also the periodic halo of u, v, w, with the
// result of pw_halo_kernel after this kernel.  A thread copies its own points
// once it has written them: the boundary planes and columns, which are in the
// cache, are read again, so that only the threads that hold them carry that
// code, its registers are not needed beside the perturbation's (59-69 in all,
// seven or eight waves per SIMD; with the copies made from the values in hand
// 123-135, three or four), and a record may give one array for several fields.
// Bound by the HBM for 4- and 8-byte storage and by instruction issue (two
// 32-bit hashes per element, whose four multiplications run at a quarter of the
// rate) for the 16-bit types: 384 domains FP64 771 us (4.5 GB, 5.8 TB/s), FP32
// 366 (VALU busy 0.53), int32 367, BF16 268 (1.05 GB, VALU busy 0.83); with the
// copies in hand and the advection's tiles as its split 773, 377, 743 and 362;
// as perturbation and halo fill one after the other 726 + 102, 351 + 81, 349 +
// 77 and 223 + 61 and a launch.  20 domains: FP64 37, FP32 22, int32 23, BF16
// 20 us (37, 24, 40, 26 and 39, 25, 26, 29).
constexpr int kPerturbPlanes = 4;

template <typename ST, bool HALO>
__global__ __launch_bounds__(256) void pw_perturb_kernel(const BatchDomain* __restrict__ table, int ndom, int chunk,
                                                         int planes, const pw_domain_args* __restrict__ args, uint64_t seed,
                                                         const unsigned long long* __restrict__ call, double amp) {
    using CT = typename compute_of<ST>::type;
    // HALO: from the last workgroup's share to the first's, so that the
    // advection after it, which begins with the first tiles, finds the fields
    // written last in the last-level cache (and so does the next step's
    // perturbation)
    const int t = HALO ? (int)(gridDim.x - 1 - blockIdx.x) : (int)blockIdx.x;
    const BatchDomain b = table[find_domain(table, ndom, t, &BatchDomain::fill_begin)];
    const int dom = b.rec;   // the caller's domain index keys the hash
    const pw_domain_args& a = args[dom];
    if (!shape_matches(a.shape, b) || !a.u || !a.v) return;
    const int local = t - b.fill_begin;
    const int c = local % b.nchunks;
    const int sg = local / b.nchunks;
    const int len = segment_split(b.nx, planes).len;
    const int i0 = 1 + sg * len;                 // <= nx: segments start at or before plane nx
    const int i1 = min(i0 + len - 1, b.nx);
    const uint32_t nz = (uint32_t)b.nz, nyz = (uint32_t)b.ny * (uint32_t)b.nz;   // nx ny nz < 2^31 (plan time)
    const uint32_t pend = min((uint32_t)(c + 1) * (uint32_t)chunk, nyz);
    const uint64_t key64 = splitmix64(seed ^ splitmix64((uint64_t)(*call) * 0x100000001b3ull + (uint64_t)dom));
    const uint32_t key = (uint32_t)key64 ^ (uint32_t)(key64 >> 32);
    using U = storage_bits<ST>;
    global_ptr<U> f[3] = {as_global((U*)a.u), as_global((U*)a.v), as_global((U*)a.w)};
    const CT sc[2] = {static_cast<CT>(scaled_type<ST>::value ? scale_or_one(a.scales.in_scale[0]) : 1.0f),
                      static_cast<CT>(scaled_type<ST>::value ? scale_or_one(a.scales.in_scale[1]) : 1.0f)};
    // x + amp r (times the field's scale) for the element whose hash index (2 g + q) is n
    auto perturbed = [&](CT x, uint32_t n, int q) {
        const uint32_t h = lowbias32(key ^ lowbias32(n));
        const float r = (float)(h >> 8) * 0x1.0p-23f - 1.0f;   // [-1, 1)
        return x + static_cast<CT>(amp * (double)r) * sc[q];
    };
    // the planes i0 .. i1 in groups of kPerturbPlanes and a remainder
    auto by_groups = [&](auto group) {
        int i = i0;
        for (; i + kPerturbPlanes - 1 <= i1; i += kPerturbPlanes) group(std::integral_constant<int, kPerturbPlanes>{}, i);
        static_assert(kPerturbPlanes == 4, "remainders of one to three planes");
        if (i + 2 == i1) group(std::integral_constant<int, 3>{}, i);
        else if (i + 1 == i1) group(std::integral_constant<int, 2>{}, i);
        else if (i == i1) group(std::integral_constant<int, 1>{}, i);
    };
    for (uint32_t p = (uint32_t)c * (uint32_t)chunk + threadIdx.x; p < pend; p += 256) {
        const uint32_t k = p % nz;
        const uint32_t j = p / nz + 1;
        const int64_t col = k + (int64_t)j * b.sy;
        const int64_t step = b.sx;   // uniform
        global_ptr<U> at[2] = {f[0] + (col + (int64_t)i0 * step), f[1] + (col + (int64_t)i0 * step)};
        uint32_t n = 2u * ((uint32_t)(i0 - 1) * nyz + p);
        // N planes: all their loads first (unconditional, so they are in flight
        // together), then the results
        auto perturb = [&](auto count, int) {
            constexpr int N = decltype(count)::value;
            CT x[N][2];
#pragma unroll
            for (int u = 0; u < N; ++u)
#pragma unroll
                for (int q = 0; q < 2; ++q) x[u][q] = to_compute(from_bits<ST>(at[q][u * step]));
#pragma unroll
            for (int u = 0; u < N; ++u)
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    at[q][u * step] = to_bits(from_compute<ST>(perturbed(x[u][q], n + 2u * (uint32_t)u * nyz + (uint32_t)q, q)));
#pragma unroll
            for (int q = 0; q < 2; ++q) at[q] += N * step;
            n += 2u * N * nyz;
        };
        by_groups(perturb);
        if (HALO && a.w != nullptr) {   // a record without a field has no halo fill
            // halo columns that copy this one (both may for ny = 1)
            const bool to_lo = (int)j == b.ny, to_hi = j == 1;
            const int64_t lo = k, hi = k + (int64_t)(b.ny + 1) * b.sy;
            // this point of plane `from` to plane `to`, and to the halo columns there
            auto plane_copy = [&](int from, int to) {
                U x[3];
#pragma unroll
                for (int q = 0; q < 3; ++q) x[q] = f[q][col + from * step];
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    f[q][col + to * step] = x[q];
                    if (to_lo) f[q][lo + to * step] = x[q];
                    if (to_hi) f[q][hi + to * step] = x[q];
                }
            };
            if (i0 == 1) plane_copy(1, b.nx + 1);
            if (i1 == b.nx) plane_copy(b.nx, 0);
            // this column to the halo columns in N planes, all loads first
            auto column_copy = [&](auto count, int i) {
                constexpr int N = decltype(count)::value;
                U x[N][3];
#pragma unroll
                for (int u = 0; u < N; ++u)
#pragma unroll
                    for (int q = 0; q < 3; ++q) x[u][q] = f[q][col + (i + u) * step];
#pragma unroll
                for (int u = 0; u < N; ++u)
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        if (to_lo) f[q][lo + (i + u) * step] = x[u][q];
                        if (to_hi) f[q][hi + (i + u) * step] = x[u][q];
                    }
            };
            if (to_lo || to_hi) {
                int i = i0;
                for (; i < i1; i += 2) column_copy(std::integral_constant<int, 2>{}, i);
                if (i == i1) column_copy(std::integral_constant<int, 1>{}, i);
            }
        }
    }
}

__global__ void pw_bump_kernel(unsigned long long* call) { *call += 1ull; }

// Everything one launch of the batched kernel needs besides the records.
struct BatchedLaunch {
    const BatchDomain* table;
    int32_t ndomains;
    int64_t tiles;
    int64_t workgroups;
    int64_t lds_bytes;
    unsigned long long* errors;
    const uint32_t* gate;
    bool vec_shapes;
    bool one_per_tile;
    const int32_t* order;   // one workgroup per tile: the plan's dispatch order, or NULL (runs of kOneTileRuns)
    unsigned long long* bump;   // counter to increment, or NULL
};

template <typename ST, int P, int KIND>
hipError_t launch_batched(const BatchedLaunch& bl, const pw_domain_args* args, hipStream_t stream) {
    auto kern = pw_batched_kernel<ST, 256, P, KIND>;
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [&] {
        attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kMaxDynamicLds);
    });
    if (attr_err != hipSuccess) return attr_err;
    hipLaunchKernelGGL(kern, dim3((unsigned)bl.workgroups), dim3(256), (size_t)bl.lds_bytes, stream, bl.table,
                       bl.ndomains, bl.tiles, args, bl.errors, bl.vec_shapes ? 1 : 0, bl.one_per_tile ? 1 : 0,
                       bl.order, bl.gate, bl.bump);
    return hipGetLastError();
}

template <typename ST, int P, int KIND>
int occupancy_of(int64_t lds_bytes) {
    int n = 0;
    auto kern = pw_batched_kernel<ST, 256, P, KIND>;
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                              kMaxDynamicLds);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kern, 256, (size_t)lds_bytes) != hipSuccess) return 0;
    return n;
}

template <typename ST, int P>
int occupancy_kind(int32_t kind, int64_t lds_bytes) {
    switch (kind) {
        case kFixedNz: return occupancy_of<ST, P, kFixedNz>(lds_bytes);
        case kEven0: return occupancy_of<ST, P, kEven0>(lds_bytes);
        case kEven1: return occupancy_of<ST, P, kEven1>(lds_bytes);
        case kEven2: return occupancy_of<ST, P, kEven2>(lds_bytes);
        case kClass0: return occupancy_of<ST, P, kClass0>(lds_bytes);
        case kClass1: return occupancy_of<ST, P, kClass1>(lds_bytes);
        case kClass2: return occupancy_of<ST, P, kClass2>(lds_bytes);
        default: return 0;
    }
}

template <typename ST>
int occupancy_typed(int32_t chunk, int32_t kind, int64_t lds_bytes) {
    switch (chunk) {
        case 256: return occupancy_kind<ST, 256>(kind, lds_bytes);
        case 512: return occupancy_kind<ST, 512>(kind, lds_bytes);
        case 1024: return occupancy_kind<ST, 1024>(kind, lds_bytes);
        default: return 0;
    }
}

// Resident workgroups per CU of the batched kernel (registers and LDS).
int batched_occupancy(int32_t storage, int32_t chunk, int32_t kind, int64_t lds_bytes) {
    switch (storage) {
        case PW_F64: return occupancy_typed<double>(chunk, kind, lds_bytes);
        case PW_F32: return occupancy_typed<float>(chunk, kind, lds_bytes);
        case PW_BF16: return occupancy_typed<bf16_t>(chunk, kind, lds_bytes);
        case PW_F16: return occupancy_typed<f16_t>(chunk, kind, lds_bytes);
        case PW_I16: return occupancy_typed<fx16_t>(chunk, kind, lds_bytes);
        case PW_I32: return occupancy_typed<fx32_t>(chunk, kind, lds_bytes);
        default: return 0;
    }
}

// Workgroups per CU of a batched launch, asked of the runtime once for each
// kernel and LDS size (the allocation-free call needs it on every call).
int64_t resident_per_cu(int32_t storage, int32_t chunk, int32_t kind, int64_t lds_bytes) {
    static std::atomic<int32_t> known[6][3][7][3];   // 0: not asked yet; kFixedNz: by its height's LDS
    const int c = chunk == 256 ? 0 : (chunk == 512 ? 1 : 2);
    const int h = kind != kFixedNz || lds_bytes == march_lds_bytes(storage, chunk, 64)
                      ? 0 : (lds_bytes == march_lds_bytes(storage, chunk, 96) ? 1 : 2);
    std::atomic<int32_t>& slot = known[storage][c][kind][h];
    int32_t occ = slot.load(std::memory_order_relaxed);
    if (occ == 0) {
        occ = batched_occupancy(storage, chunk, kind, lds_bytes);
        if (occ > 0) slot.store(occ, std::memory_order_relaxed);
    }
    const int64_t by_lds = std::max<int64_t>(1, kLdsPerCu / std::max<int64_t>(lds_bytes, 1));
    const int64_t n = std::min<int64_t>(by_lds, 8);
    return occ > 0 ? std::min<int64_t>(n, occ) : n;
}

// Default segment length of a batch from its chunk planes and the workgroups
// the chip keeps resident: 1.3 times the chunk planes per resident workgroup,
// so that a small batch still gives every CU tiles of equal length, at least
// 6 (below, the planes a tile's start reads twice cost more than the balance
// gains) and at most the length that is best for large batches: 10 planes for
// FP64 and 12 for FP32, where short tiles keep the uneven domains' streams
// together in HBM.  Fitted to lengths of 1 .. 96 planes on batches of 5 to 384
// domains: on average 1.6% (FP64) and 2.7% (FP32) off the best length; fixed
// lengths of 16 planes are 9% and 13% off.  384 domains FP64 1114 -> 1087 us.
// The types that convert (scheduled_seg with a plan) take 0.7 times the chunk
// planes per workgroup, at most 48 planes, where nothing orders the tiles by
// length: 96 domains BF16 106 us with 32 planes, 112 with 64; 30 domains 43
// with 16, 53 with 64.
int32_t batched_seg(int32_t storage, int64_t planes, int64_t resident) {
    const bool wide = storage == PW_F64 || storage == PW_F32;
    const int64_t most = storage == PW_F64 ? 10 : (wide ? 12 : 48);
    const int64_t seg = planes * (wide ? 13 : 7) / (10 * std::max<int64_t>(1, resident));
    return (int32_t)std::max<int64_t>(6, std::min<int64_t>(seg, most));
}

// Dispatch order of a plan's one-workgroup-per-tile launch.  Each domain's
// chunks form groups of kOneTileRuns neighbours (they share y-halo columns),
// and every segment of a group runs on one XCD; the groups are spread over
// the XCDs by their points, the longest tiles first.  An XCD's queue takes
// its groups in windows of about as many tiles as the XCD keeps resident
// and runs segment 0 of every group of the window, then segment 1, and so on
// -- the march kernel's compact order within each window -- so the tile of
// segment s + 1 of a group starts as the window's segment-s tiles retire and
// finds the planes they share still in the XCD's L2.  Workgroups go
// round-robin over the XCDs: order[k * 8 + x] is the tile of the k-th
// workgroup of XCD x, -1 past the end of that XCD's queue.
struct Group {
    int d, c0, c1;
};
std::vector<std::vector<Group>> xcd_groups(const std::vector<BatchDomain>& table) {
    std::vector<std::vector<Group>> groups(kNumXcd);
    std::vector<int64_t> load(kNumXcd, 0);
    for (int d = 0; d < (int)table.size(); ++d) {
        const BatchDomain& b = table[d];
        for (int c0 = 0; c0 < b.nchunks; c0 += kOneTileRuns) {
            const int c1 = std::min(b.nchunks, c0 + kOneTileRuns);
            const int x = (int)(std::min_element(load.begin(), load.end()) - load.begin());
            groups[x].push_back(Group{d, c0, c1});
            load[x] += (int64_t)(c1 - c0) * b.nx;
        }
    }
    return groups;
}
// f(group, segment) in an XCD's queue order.
template <typename F>
void in_windows(const std::vector<BatchDomain>& table, const std::vector<Group>& gs, int64_t resident_per_xcd, F f) {
    const size_t window = (size_t)std::max<int64_t>(1, resident_per_xcd / kOneTileRuns);   // groups in flight
    for (size_t w0 = 0; w0 < gs.size(); w0 += window) {
        const size_t w1 = std::min(gs.size(), w0 + window);
        int nseg = 0;
        for (size_t i = w0; i < w1; ++i) nseg = std::max(nseg, table[gs[i].d].nseg);
        for (int sg = 0; sg < nseg; ++sg)
            for (size_t i = w0; i < w1; ++i)
                if (sg < table[gs[i].d].nseg) f(gs[i], sg);
    }
}
std::vector<int32_t> one_tile_order(const std::vector<BatchDomain>& table, int64_t resident_per_xcd) {
    const std::vector<std::vector<Group>> groups = xcd_groups(table);
    std::vector<std::vector<int32_t>> queue(kNumXcd);
    for (int x = 0; x < kNumXcd; ++x)
        in_windows(table, groups[x], resident_per_xcd, [&](const Group& g, int sg) {
            const BatchDomain& b = table[g.d];
            for (int c = g.c0; c < g.c1; ++c)
                queue[x].push_back((int32_t)(b.tile_begin + (int64_t)sg * b.nchunks + c));
        });
    size_t len = 0;
    for (const std::vector<int32_t>& q : queue) len = std::max(len, q.size());
    std::vector<int32_t> order(len * kNumXcd, -1);
    for (int x = 0; x < kNumXcd; ++x)
        for (size_t k = 0; k < queue[x].size(); ++k) order[k * kNumXcd + x] = queue[x][k];
    return order;
}

// Default segment length of a plan's batch for the types that convert, whose
// tiles' start costs more, so that longer tiles and the rounds they fill
// matter: the length with the least predicted time.  The tiles, longest first
// (`grouped`: in the XCDs' queues), go to the resident workgroups as those come
// free (a tile of n planes takes n + 3 plane steps); 0.7 of the time are the
// mean workgroup's steps and 0.3 the last one's, since the chip's rate falls
// less than the workgroups left.  Lengths: 1.3 times the chunk planes per
// resident workgroup, and from half to twice the chunk planes.  Measured on 54
// batches of 10 to 90 domains over all of these lengths: 1.4% (int32), 1.1%
// (BF16) and 0.7% (int16) off the best length on average; 1.3 times alone, 5%, 8% and 5%, because it fills one and a
// bit rounds as often as two (30 domains int32 62 us with 49 planes, 50 with
// 56; 45 domains int16 54 with 64, 50 with 27); one length for every batch (16
// planes for int32, 64 for the others), 12%, 44% and 47%.  Batches of more than
// 128 chunk planes per resident workgroup take 64 planes (384 domains int32
// 632 us, with 16 planes 710).
int32_t scheduled_seg(const pw_shape* shapes, int32_t n, int32_t chunk, int64_t planes, int64_t resident, bool grouped) {
    constexpr int64_t kBegin = 3;
    const int64_t slots = std::max<int64_t>(kNumXcd, resident);
    if (planes > 128 * slots) return 64;
    std::vector<BatchDomain> rows(n);
    std::vector<int64_t> at;   // workgroups that come free at each step
    size_t now = 0, end = 0;
    auto begin = [&](int64_t workgroups, int64_t steps, int32_t longest) {
        // no tile starts after the mean workgroup's end
        at.assign((size_t)(steps / workgroups + longest + kBegin + 1), 0);
        at[0] = workgroups;
        now = 0;
    };
    auto run = [&](int64_t tiles, int32_t len) {
        while (tiles > 0) {
            while (at[now] == 0) ++now;
            const int64_t m = std::min(tiles, at[now]);
            const size_t done = now + (size_t)(len + kBegin);
            at[now] -= m;
            at[done] += m;
            tiles -= m;
            end = std::max(end, done);
        }
    };
    auto length = [](const BatchDomain& b, int sg) { return sg + 1 < b.nseg ? b.seg : b.nx - b.seg * (b.nseg - 1); };
    auto predicted = [&](int32_t most) {
        int64_t steps = 0;
        for (int32_t d = 0; d < n; ++d) {
            domain_tiles(shapes[d].nx, shapes[d].ny, shapes[d].nz, chunk, most, &rows[d]);
            steps += (int64_t)rows[d].nchunks * (rows[d].nx + kBegin * rows[d].nseg);
        }
        std::stable_sort(rows.begin(), rows.end(), [](const BatchDomain& x, const BatchDomain& y) { return x.seg > y.seg; });
        end = 0;
        if (grouped) {
            for (const std::vector<Group>& gs : xcd_groups(rows)) {
                int64_t own = 0;
                for (const Group& g : gs) own += (int64_t)(g.c1 - g.c0) * (rows[g.d].nx + kBegin * rows[g.d].nseg);
                begin(slots / kNumXcd, own, most);
                in_windows(rows, gs, slots / kNumXcd, [&](const Group& g, int sg) { run(g.c1 - g.c0, length(rows[g.d], sg)); });
            }
        } else {
            begin(slots, steps, most);
            for (const BatchDomain& b : rows) {
                run((int64_t)b.nchunks * (b.nseg - 1), b.seg);
                run(b.nchunks, length(b, b.nseg - 1));
            }
        }
        return 0.3 * (double)end + 0.7 * (double)steps / (double)slots;
    };
    int32_t best = (int32_t)std::max<int64_t>(6, std::min<int64_t>(planes * 13 / (10 * slots), 64));
    double least = predicted(best);
    for (int32_t most = 6; most <= 64; most += std::max(1, most / 8)) {   // .., 16, 18, .., 51, 57, 64
        if (2 * most * slots < planes || most * slots > 2 * planes) continue;
        const double t = predicted(most);
        if (t < least) {
            least = t;
            best = most;
        }
    }
    return best;
}

template <typename ST, int P>
hipError_t dispatch_kind(int32_t kind, const BatchedLaunch& bl, const pw_domain_args* args, hipStream_t stream) {
    switch (kind) {
        case kFixedNz: return launch_batched<ST, P, kFixedNz>(bl, args, stream);
        case kEven0: return launch_batched<ST, P, kEven0>(bl, args, stream);
        case kEven1: return launch_batched<ST, P, kEven1>(bl, args, stream);
        case kEven2: return launch_batched<ST, P, kEven2>(bl, args, stream);
        case kClass0: return launch_batched<ST, P, kClass0>(bl, args, stream);
        case kClass1: return launch_batched<ST, P, kClass1>(bl, args, stream);
        case kClass2: return launch_batched<ST, P, kClass2>(bl, args, stream);
        default: return hipErrorInvalidValue;
    }
}

template <typename ST>
hipError_t dispatch_chunk(int32_t chunk, int32_t kind, const BatchedLaunch& bl, const pw_domain_args* args,
                          hipStream_t stream) {
    switch (chunk) {
        case 256: return dispatch_kind<ST, 256>(kind, bl, args, stream);
        case 512: return dispatch_kind<ST, 512>(kind, bl, args, stream);
        case 1024: return dispatch_kind<ST, 1024>(kind, bl, args, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t dispatch_batched(int32_t storage, int32_t chunk, int32_t kind, const BatchedLaunch& bl,
                            const pw_domain_args* args, hipStream_t stream) {
    switch (storage) {
        case PW_F64: return dispatch_chunk<double>(chunk, kind, bl, args, stream);
        case PW_F32: return dispatch_chunk<float>(chunk, kind, bl, args, stream);
        case PW_BF16: return dispatch_chunk<bf16_t>(chunk, kind, bl, args, stream);
        case PW_F16: return dispatch_chunk<f16_t>(chunk, kind, bl, args, stream);
        case PW_I16: return dispatch_chunk<fx16_t>(chunk, kind, bl, args, stream);
        case PW_I32: return dispatch_chunk<fx32_t>(chunk, kind, bl, args, stream);
        default: return hipErrorInvalidValue;
    }
}

// Workgroups per domain of the halo fill: the mean domain's halo in blocks
// of 256 elements (larger domains loop), at most the largest domain's and a
// million.
int64_t halo_blocks(const pw_plan* p) {
    int64_t m = 0, sum = 0;
    for (const pw_shape& s : p->shapes) {
        const int64_t e = halo_columns(s.nx, s.ny) * s.nz;
        m = std::max<int64_t>(m, e);
        sum += e;
    }
    const int64_t mean = sum / std::max<int64_t>(1, (int64_t)p->shapes.size());
    return std::max<int64_t>(1, std::min<int64_t>({(m + 255) / 256, (mean + 255) / 256, int64_t(1) << 20}));
}

}  // namespace

// Tile split of one domain: nchunks chunks of `chunk` points per plane, x
// range split into nseg segments of even length (at most seg_max planes).
__host__ __device__ inline void domain_tiles(int32_t nx, int32_t ny, int32_t nz, int32_t chunk, int32_t seg_max,
                                             BatchDomain* b) {
    b->nx = nx;
    b->ny = ny;
    b->nz = nz;
    b->nchunks = (int32_t)(((int64_t)ny * nz + chunk - 1) / chunk);
    const SegmentSplit x = segment_split(nx, seg_max);
    b->nseg = x.n;
    b->seg = x.len;
}

// Launch shape of the batched kernel for a list of (normalised) shapes:
// chunk, segment bound, LDS, code-path kind, total tiles and grid.  Allocates
// nothing.  Returns PW_OK with L->tiles == 0 if a shape cannot use the
// batched kernel (march variant impossible, or 2^31 points or more).
int32_t batched_launch_shape(int32_t storage, const pw_shape* shapes, int32_t n, const pw_tuning& t, Launch* L,
                             int32_t* kind, bool* vec_out, bool sorted) {
    *L = Launch{};
    for (int32_t d = 0; d < n; ++d) {
        pw_shape s;
        const int32_t rc = normalize_shape(shapes[d], &s);
        if (rc != PW_OK) return rc;
        if (!march_possible(s) || (int64_t)s.nx * s.ny * s.nz >= (int64_t(1) << 31)) return PW_OK;
    }
    const int32_t chunk = t.chunk ? t.chunk : 512;
    if (chunk != 256 && chunk != 512 && chunk != 1024) return PW_ERR_INVALID_ARG;
    if (t.seg < 0 || t.wg_per_cu < PW_WG_ONE_PER_TILE || t.wg_per_cu > 8) return PW_ERR_INVALID_ARG;
    int32_t nzmax = 0;
    int64_t planes = 0;   // chunk planes of the batch
    bool vec = true, fixed_nz = true, even = true;
    for (int32_t d = 0; d < n; ++d) {
        pw_shape s;
        (void)normalize_shape(shapes[d], &s);   // checked above
        planes += ((int64_t)s.ny * s.nz + chunk - 1) / chunk * s.nx;
        nzmax = std::max(nzmax, s.nz);
        vec = vec && vector_shape(storage, s);
        fixed_nz = fixed_nz && compiled_height(s.nz);
        even = even && s.nz % 2 == 0;
    }
    Launch r{};
    r.variant = PW_VARIANT_MARCH;
    r.chunk = chunk;
    r.block = 256;
    const int32_t k = vec && fixed_nz ? kFixedNz : (even ? kEven0 : kClass0) + height_class(nzmax);
    r.lds_bytes = march_lds_bytes(storage, chunk, k == kFixedNz ? nzmax : -kHeightClass[kind_class(k)]);
    if (r.lds_bytes > kMaxDynamicLds) return PW_ERR_UNSUPPORTED;
    int dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return report_hip(e);
    int64_t per_cu = resident_per_cu(storage, chunk, k, r.lds_bytes);
    const int64_t resident = (int64_t)cus * std::min<int64_t>(per_cu, 4);
    r.seg = t.seg ? t.seg
                  : (sorted && storage != PW_F64 && storage != PW_F32
                         ? scheduled_seg(shapes, n, chunk, planes, resident, storage == PW_BF16 || storage == PW_F16)
                         : batched_seg(storage, planes, resident));
    auto count = [&] {
        int64_t tiles = 0;
        for (int32_t d = 0; d < n; ++d) {
            BatchDomain b{};
            domain_tiles(shapes[d].nx, shapes[d].ny, shapes[d].nz, chunk, r.seg, &b);
            tiles += (int64_t)b.nchunks * b.nseg;
        }
        return tiles;
    };
    int64_t tiles = count();
    // a default segment length never makes more tiles than a launch may hold
    // (unless whole domains do)
    while (!t.seg && tiles > kMaxTiles && r.seg < (1 << 30)) {
        r.seg *= 2;
        tiles = count();
    }
    r.tiles = tiles;
    if (t.wg_per_cu > 0) per_cu = std::min<int64_t>(per_cu, t.wg_per_cu);
    r.workgroups = std::max<int64_t>(1, std::min<int64_t>(tiles, (int64_t)cus * per_cu));
    // One workgroup per tile: the kernel's tile loop then runs once per
    // workgroup, and the hardware dispatches tiles in order as workgroups
    // retire, so the workgroups on neighbouring chunks stay in step (their
    // shared halo columns meet in L2) where a persistent grid's fixed
    // round-robin shares drift apart.  Measured on the 384-domain batch: 2-3%
    // faster than the best persistent grid for FP64, FP32 and BF16, and 11-18%
    // faster than a persistent grid at full occupancy; hence the default.
    if (batched_one_per_tile(t)) {
        constexpr int64_t block = (int64_t)kNumXcd * kOneTileRuns;   // padded to whole blocks (kernel comment)
        const int64_t g = (tiles + block - 1) / block * block;
        if (g >= (int64_t(1) << 31)) return PW_ERR_UNSUPPORTED;
        r.workgroups = g;
    }
    *L = r;
    *kind = k;
    *vec_out = vec;
    return PW_OK;
}

// The perturbation's split of a batch (its rows' fill_begin): most planes of a
// workgroup and, in *fill_tiles, the workgroups; `planes` chunk planes in all.
// Enough workgroups for two rounds of a full chip (eight workgroups per CU), at
// least 6 planes (below, finding its domain costs a workgroup more than the
// balance gains) and at most 10.  With 6, 10, 16, 24, 40 and 64 planes, recorded
// timesteps of 12 domains FP64 68, 69, 71, 74, 79, 85 us; of 60 domains BF16 97,
// 96, 97, 100, 104, 112, int32 145, 145, 146, 147, 154, 164; of 384, FP32 947,
// 953, 959, 965, 974, 983, int16 606, 585, 577, 575, 582, 601.
int32_t fill_split(std::vector<BatchDomain>& table, int64_t planes, int cus, int64_t* fill_tiles) {
    int64_t most = std::max<int64_t>(6, std::min<int64_t>(planes / (16 * (int64_t)cus), 10));
    for (;; most *= 2) {
        int64_t t = 0;
        for (const BatchDomain& b : table) t += (int64_t)b.nchunks * segment_split(b.nx, (int32_t)most).n;
        *fill_tiles = t <= kMaxTiles ? t : 0;
        if (t <= kMaxTiles || most >= (1 << 30)) break;   // a launch holds them, or none can
    }
    int64_t at = 0;
    for (BatchDomain& b : table) {
        b.fill_begin = (int32_t)at;
        at += (int64_t)b.nchunks * segment_split(b.nx, (int32_t)most).n;
    }
    return (int32_t)most;
}

int32_t batched_plan_init(pw_plan* p) {
    BatchState& B = p->batch;
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(nullptr, &cs) == hipSuccess && cs != hipStreamCaptureStatusNone) return PW_ERR_CAPTURE;
    Launch L{};
    int32_t kind = kFixedNz;
    bool vec = false;
    int32_t rc = batched_launch_shape(p->storage, p->shapes.data(), p->ndomains, p->tuning, &L, &kind, &vec,
                                      batched_one_per_tile(p->tuning));
    if (rc != PW_OK) return rc;
    if (L.tiles == 0) return PW_OK;   // batched entry points will report PW_ERR_UNSUPPORTED

    std::vector<BatchDomain> rows(p->ndomains);
    for (int32_t d = 0; d < p->ndomains; ++d) {
        const pw_shape& s = p->shapes[d];
        BatchDomain& b = rows[d];
        domain_tiles(s.nx, s.ny, s.nz, L.chunk, L.seg, &b);
        b.sy = s.sy;
        b.sx = s.sx;
        b.rec = d;
    }
    // One workgroup per tile: longest tiles first (stable: equal lengths keep
    // the caller's order), so long tiles start early and short ones fill the
    // end.  A persistent grid keeps the caller's order: its XCDs walk
    // contiguous shares of the list, which a sorted list would leave
    // unbalanced (measured 9-16% slower on the 384-domain batch).
    if (batched_one_per_tile(p->tuning))
        std::stable_sort(rows.begin(), rows.end(),
                         [](const BatchDomain& x, const BatchDomain& y) { return x.seg > y.seg; });
    std::vector<BatchDomain>& table = rows;
    int64_t tiles = 0, planes = 0;
    for (BatchDomain& b : table) {
        b.tile_begin = tiles;
        tiles += (int64_t)b.nchunks * b.nseg;
        planes += (int64_t)b.nchunks * b.nx;
    }
    int dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return report_hip(e);
    B.fill_planes = fill_split(table, planes, cus, &B.fill_tiles);
    std::vector<int32_t> order;
    // The grouped order (one_tile_order) measured 6-11% faster than runs of
    // kOneTileRuns for BF16 and FP16 batches, whose kernels are bound by
    // instruction issue and gain from the L2 hits; 4-7% slower for FP64 and
    // FP32, bound by HBM, which gain more from all XCDs streaming neighbouring
    // tiles of the list at once, and 0.5-1% slower for int16.  So only BF16
    // and FP16 use it.
    if (batched_one_per_tile(p->tuning) && (p->storage == PW_BF16 || p->storage == PW_F16) &&
        tiles < (int64_t(1) << 31)) {
        // workgroups one XCD keeps resident: its CUs times the occupancy
        const int64_t per_cu = resident_per_cu(p->storage, L.chunk, kind, L.lds_bytes);
        order = one_tile_order(table, std::max<int64_t>(1, cus / kNumXcd) * per_cu);
        if ((int64_t)order.size() > kMaxTiles) order.clear();   // one long queue: the grid would not fit a launch
        if (!order.empty()) L.workgroups = (int64_t)order.size();
    }
    void* mem = nullptr;
    const size_t tbytes = sizeof(BatchDomain) * table.size();
    // one allocation: the tile table, the error count, then the dispatch order
    const size_t off_err = (tbytes + 63) / 64 * 64;
    const size_t off_order = off_err + 64;
    e = hipMalloc(&mem, off_order + sizeof(int32_t) * order.size());
    if (e == hipErrorOutOfMemory) return PW_ERR_OUT_OF_MEMORY;
    if (e != hipSuccess) return report_hip(e);
    B.d_table = static_cast<BatchDomain*>(mem);
    B.d_errors = reinterpret_cast<unsigned long long*>(static_cast<char*>(mem) + off_err);
    B.d_order = order.empty() ? nullptr : reinterpret_cast<const int32_t*>(static_cast<char*>(mem) + off_order);
    e = hipMemcpy(B.d_table, table.data(), tbytes, hipMemcpyHostToDevice);
    if (e == hipSuccess && !order.empty())
        e = hipMemcpy(static_cast<char*>(mem) + off_order, order.data(), sizeof(int32_t) * order.size(),
                      hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemset(B.d_errors, 0, sizeof(unsigned long long));
    if (e == hipSuccess) e = hipStreamSynchronize(nullptr);   // zeroed before any launch on another stream
    if (e != hipSuccess) {
        (void)hipFree(mem);
        B.d_table = nullptr;
        B.d_errors = nullptr;
        B.d_order = nullptr;
        return report_hip(e);
    }
    B.launch = L;
    B.device = dev;
    B.vec_shapes = vec;
    B.kind = kind;
    return PW_OK;
}

int32_t batched_plan_free(pw_plan* p) {
    if (p->batch.d_table) {
        hipError_t e = hipFree(p->batch.d_table);
        p->batch.d_table = nullptr;
        p->batch.d_errors = nullptr;
        p->batch.d_order = nullptr;
        if (e != hipSuccess) return report_hip(e);
    }
    return PW_OK;
}

// The advection of a batch; `bump` (or NULL): a counter the launch increments.
static int32_t launch_advect(const pw_plan* plan, const pw_domain_args* d_args, unsigned long long* bump, hipStream_t s) {
    const BatchState& B = plan->batch;
    const BatchedLaunch bl{B.d_table, plan->ndomains, B.launch.tiles, B.launch.workgroups, B.launch.lds_bytes,
                           B.d_errors, nullptr, B.vec_shapes, batched_one_per_tile(plan->tuning),
                           B.d_order, bump};
    const hipError_t e = dispatch_batched(plan->storage, B.launch.chunk, B.kind, bl, d_args, s);
    return e == hipSuccess ? PW_OK : report_hip(e);
}

// The perturbation of a batch (HALO: and its halo fill).
template <bool HALO>
static int32_t launch_perturb(const pw_plan* plan, const pw_domain_args* d_args, uint64_t seed,
                              const unsigned long long* d_call, double amplitude, hipStream_t s) {
    const BatchState& B = plan->batch;
    if (B.fill_tiles == 0) return PW_ERR_UNSUPPORTED;
    const dim3 grid((unsigned)B.fill_tiles);
    const BatchDomain* tb = B.d_table;
    const int nd = plan->ndomains, ch = B.launch.chunk, planes = B.fill_planes;
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, tb, nd, ch, planes, d_args, seed, d_call, amplitude);
        return hipGetLastError();
    };
    hipError_t e = hipSuccess;
    switch (plan->storage) {
        case PW_F64: e = go(pw_perturb_kernel<double, HALO>); break;
        case PW_F32: e = go(pw_perturb_kernel<float, HALO>); break;
        case PW_BF16: e = go(pw_perturb_kernel<bf16_t, HALO>); break;
        case PW_F16: e = go(pw_perturb_kernel<f16_t, HALO>); break;
        case PW_I16: e = go(pw_perturb_kernel<fx16_t, HALO>); break;
        case PW_I32: e = go(pw_perturb_kernel<fx32_t, HALO>); break;
        default: return PW_ERR_UNSUPPORTED;
    }
    return e == hipSuccess ? PW_OK : report_hip(e);
}

// One timestep in two launches: perturbation with the halo fill, then the
// advection, which also advances the call counter (the next step's
// perturbation reads it after this launch).
int32_t record_timestep(const pw_plan* plan, const pw_domain_args* d_args, uint64_t seed, unsigned long long* d_call,
                        double amplitude, hipStream_t s) {
    const int32_t rc = launch_perturb<true>(plan, d_args, seed, d_call, amplitude, s);
    return rc == PW_OK ? launch_advect(plan, d_args, d_call, s) : rc;
}

}  // namespace pw

using namespace pw;

extern "C" {

int32_t pw_advect_batched(const pw_plan* plan, int32_t ndomains, const pw_domain_args* d_args, void* stream) {
    if (!plan || !d_args) return PW_ERR_INVALID_ARG;
    if (ndomains != plan->ndomains) return PW_ERR_PLAN_MISMATCH;
    if (!plan->batch.d_table) return PW_ERR_UNSUPPORTED;
    if (elem_bytes(plan->storage) == 0) return PW_ERR_UNSUPPORTED;
    return launch_advect(plan, d_args, nullptr, static_cast<hipStream_t>(stream));
}

int32_t pw_fill_halo_batched(const pw_plan* plan, int32_t ndomains, const pw_domain_args* d_args, void* stream) {
    if (!plan || !d_args) return PW_ERR_INVALID_ARG;
    if (ndomains != plan->ndomains) return PW_ERR_PLAN_MISMATCH;
    if (!plan->batch.d_table) return PW_ERR_UNSUPPORTED;
    dim3 grid((unsigned)halo_blocks(plan), (unsigned)ndomains);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const BatchDomain* tb = plan->batch.d_table;
    switch (plan->storage) {
        case PW_F64: hipLaunchKernelGGL(pw_halo_kernel<double>, grid, dim3(256), 0, s, tb, d_args); break;
        case PW_F32: hipLaunchKernelGGL(pw_halo_kernel<float>, grid, dim3(256), 0, s, tb, d_args); break;
        case PW_BF16: hipLaunchKernelGGL(pw_halo_kernel<bf16_t>, grid, dim3(256), 0, s, tb, d_args); break;
        case PW_F16: hipLaunchKernelGGL(pw_halo_kernel<f16_t>, grid, dim3(256), 0, s, tb, d_args); break;
        case PW_I16: hipLaunchKernelGGL(pw_halo_kernel<fx16_t>, grid, dim3(256), 0, s, tb, d_args); break;
        case PW_I32: hipLaunchKernelGGL(pw_halo_kernel<fx32_t>, grid, dim3(256), 0, s, tb, d_args); break;
        default: return PW_ERR_UNSUPPORTED;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return report_hip(e);
    return PW_OK;
}

int32_t pw_perturb_batched(const pw_plan* plan, int32_t ndomains, const pw_domain_args* d_args, uint64_t seed,
                           unsigned long long* d_call, double amplitude, void* stream) {
    if (!plan || !d_args || !d_call || !std::isfinite(amplitude)) return PW_ERR_INVALID_ARG;
    if (ndomains != plan->ndomains) return PW_ERR_PLAN_MISMATCH;
    if (!plan->batch.d_table) return PW_ERR_UNSUPPORTED;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int32_t rc = launch_perturb<false>(plan, d_args, seed, d_call, amplitude, s);
    if (rc != PW_OK) return rc;
    hipLaunchKernelGGL(pw_bump_kernel, dim3(1), dim3(1), 0, s, d_call);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return report_hip(e);
    return PW_OK;
}

int32_t pw_plan_error_count(const pw_plan* plan, unsigned long long* count) {
    if (!plan || !count) return PW_ERR_INVALID_ARG;
    *count = 0;
    if (!plan->batch.d_errors) return PW_OK;
    hipError_t e = hipMemcpy(count, plan->batch.d_errors, sizeof(unsigned long long), hipMemcpyDeviceToHost);
    if (e != hipSuccess) return report_hip(e);
    return PW_OK;
}

// ---------------------------------------------------------------------------
// Allocation-free batched call.  The tile table and the error word live in
// `scratch`, one array per GPU (file scope, allocated with the code object);
// a small kernel builds the table from the device records on every call.
// ---------------------------------------------------------------------------
}  // extern "C"

namespace pw {
namespace {

constexpr int kNoAllocMaxDomains = 4096;
constexpr int kNoAllocHeader = 64;   // gate word, tile count, error word
constexpr size_t kNoAllocScratchBytes = kNoAllocHeader + sizeof(BatchDomain) * kNoAllocMaxDomains;   // 229,440 B
static_assert(kNoAllocScratchBytes == 229440, "scratch size stated in the header");
constexpr int kMaxDevices = 64;

static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

struct ScratchSlot {
    std::once_flag once;
    hipError_t err = hipSuccess;
    unsigned char* ptr = nullptr;   // device address of this GPU's scratch
};
ScratchSlot g_scratch[kMaxDevices];

// Device address of the current GPU's `scratch`, looked up once per device
// (with that device current).  The host-side symbol is only a stand-in for
// the device array and must never be passed to a kernel or a copy.
int32_t scratch_of_current_device(unsigned char** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return report_hip(e);
    if (dev < 0 || dev >= kMaxDevices) return PW_ERR_UNSUPPORTED;
    ScratchSlot& sl = g_scratch[dev];
    std::call_once(sl.once, [&] {
        void* p = nullptr;
        sl.err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        sl.ptr = static_cast<unsigned char*>(p);
    });
    if (sl.err != hipSuccess) return report_hip(sl.err);
    if (!sl.ptr) return PW_ERR_HIP;
    *out = sl.ptr;
    return PW_OK;
}

// One term of the shape digest: a hash of (domain index, normalised shape).
// The digest of a batch is the sum of its terms (mod 2^64), so the device can
// form it with a parallel reduction and compare it with the host's.
__host__ __device__ inline uint64_t shape_digest_term(int32_t d, int32_t nx, int32_t ny, int32_t nz, int32_t reserved,
                                                      int64_t sy, int64_t sx) {
    uint64_t h = splitmix64(((uint64_t)(uint32_t)d << 32) ^ (uint64_t)(uint32_t)nx);
    h = splitmix64(h ^ (uint64_t)(uint32_t)ny);
    h = splitmix64(h ^ ((uint64_t)(uint32_t)nz | ((uint64_t)(uint32_t)reserved << 32)));
    h = splitmix64(h ^ (uint64_t)sy);
    return splitmix64(h ^ (uint64_t)sx);
}

constexpr int kTableThreads = 1024;

// Table row of domain d from its record (an empty row if the shape is out of
// range: the digest of such a batch cannot match a valid one).
__device__ __forceinline__ BatchDomain record_row(const pw_domain_args* args, int d, int chunk, int seg_max,
                                                  uint64_t* term) {
    const pw_shape s = args[d].shape;
    const int64_t sy = s.sy ? s.sy : s.nz;
    const int64_t sx = s.sx ? s.sx : (int64_t)(s.ny + 2) * sy;
    *term = shape_digest_term(d, s.nx, s.ny, s.nz, s.reserved, sy, sx);
    BatchDomain b{};
    if (s.nx >= 1 && s.ny >= 1 && s.nz >= 2 && s.nx <= (1 << 30) && (int64_t)s.ny * s.nz < (int64_t(1) << 31))
        domain_tiles(s.nx, s.ny, s.nz, chunk, seg_max, &b);
    b.sy = sy;
    b.sx = sx;
    return b;
}

// Builds the tile table of a batch from its device records into scratch (one
// workgroup of as many waves as the batch needs, at most 16): in rounds of one
// domain per thread, a scan of the tile counts (within each wave by lane
// exchange, then over the waves) gives every domain its first tile, and the
// shape digest is summed the same way.  The gate word is set only if the
// digest and the tile total equal the host's, i.e. the records carry the
// shapes the launch was shaped for.  The error word is cleared.  Bound by the
// latency of the record reads and of one launch: 8.9 us with 1024 threads of
// four domains each (two passes over the records, twenty barriers).
__global__ __launch_bounds__(kTableThreads) void pw_noalloc_table_kernel(const pw_domain_args* __restrict__ args,
                                                                         int ndom, int chunk, int seg_max,
                                                                         uint64_t digest_host, int64_t tiles_host,
                                                                         unsigned char* scr) {
    __shared__ int64_t part[kTableThreads / 64];
    __shared__ uint64_t hsum[kTableThreads / 64];
    BatchDomain* table = reinterpret_cast<BatchDomain*>(scr + kNoAllocHeader);
    const int t = (int)threadIdx.x, lane = t % 64, wave = t / 64, waves = (int)blockDim.x / 64;
    int64_t before = 0;    // tiles of the earlier rounds
    uint64_t digest = 0;   // digest terms of this thread's domains
    for (int d0 = 0; d0 < ndom; d0 += (int)blockDim.x) {   // uniform over the workgroup
        const int d = d0 + t;
        BatchDomain b{};
        if (d < ndom) {
            uint64_t term;
            b = record_row(args, d, chunk, seg_max, &term);
            digest += term;
        }
        const int64_t mine = (int64_t)b.nchunks * b.nseg;
        int64_t sum = mine;   // inclusive scan over the wave
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int64_t lower = __shfl_up(sum, off, 64);
            if (lane >= off) sum += lower;
        }
        if (lane == 63) part[wave] = sum;
        __syncthreads();
        int64_t first = before + sum - mine, all = 0;
        for (int w = 0; w < waves; ++w) {
            if (w < wave) first += part[w];
            all += part[w];
        }
        before += all;
        if (d < ndom) {
            b.rec = d;   // the caller's order (no reordering on the device)
            b.tile_begin = first;
            table[d] = b;
        }
        __syncthreads();   // part is written again in the next round
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) digest += __shfl_down(digest, off, 64);
    if (lane == 0) hsum[wave] = digest;
    __syncthreads();
    if (t == 0) {
        uint64_t h = 0;
        for (int w = 0; w < waves; ++w) h += hsum[w];
        const bool ok = h == digest_host && before == tiles_host;
        *reinterpret_cast<int64_t*>(scr + 8) = before;
        *reinterpret_cast<unsigned long long*>(scr + 16) = 0ull;
        *reinterpret_cast<uint32_t*>(scr) = ok ? 1u : 0u;
    }
}

}  // namespace
}  // namespace pw

extern "C" {

int32_t pw_advect_batched_noalloc(int32_t storage, const pw_shape* shapes, int32_t ndomains,
                                  const pw_domain_args* d_args, const pw_tuning* tuning,
                                  unsigned long long* d_skipped, void* stream) {
    if (!shapes || !d_args || ndomains < 1) return PW_ERR_INVALID_ARG;
    if (ndomains > kNoAllocMaxDomains) return PW_ERR_INVALID_ARG;
    if (elem_bytes(storage) == 0) return PW_ERR_UNSUPPORTED;
    const pw_tuning t = tuning ? *tuning : pw_tuning{};
    if (t.variant != PW_VARIANT_AUTO && t.variant != PW_VARIANT_MARCH) return PW_ERR_UNSUPPORTED;
    // digest of the normalised shapes, then the launch shape; nothing here allocates
    uint64_t digest = 0;
    for (int32_t d = 0; d < ndomains; ++d) {
        pw_shape s;
        int32_t rc = normalize_shape(shapes[d], &s);
        if (rc != PW_OK) return rc;
        digest += shape_digest_term(d, s.nx, s.ny, s.nz, s.reserved, s.sy, s.sx);
    }
    Launch L{};
    int32_t kind = 0;
    bool vec = false;
    int32_t rc = batched_launch_shape(storage, shapes, ndomains, t, &L, &kind, &vec, false);
    if (rc != PW_OK) return rc;
    if (L.tiles == 0) return PW_ERR_UNSUPPORTED;
    unsigned char* scr = nullptr;
    rc = scratch_of_current_device(&scr);
    if (rc != PW_OK) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int table_threads = std::min(kTableThreads, (ndomains + 63) / 64 * 64);   // whole waves
    hipLaunchKernelGGL(pw_noalloc_table_kernel, dim3(1), dim3((unsigned)table_threads), 0, st, d_args, ndomains, L.chunk,
                       L.seg, digest, L.tiles, scr);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return report_hip(e);
    unsigned long long* errors = d_skipped ? d_skipped : reinterpret_cast<unsigned long long*>(scr + 16);
    const BatchedLaunch bl{reinterpret_cast<const BatchDomain*>(scr + kNoAllocHeader), ndomains, L.tiles,
                           L.workgroups, L.lds_bytes, errors, reinterpret_cast<const uint32_t*>(scr), vec,
                           batched_one_per_tile(t), nullptr, nullptr};
    e = dispatch_batched(storage, L.chunk, kind, bl, d_args, st);
    if (e != hipSuccess) return report_hip(e);
    return PW_OK;
}

}  // extern "C"
