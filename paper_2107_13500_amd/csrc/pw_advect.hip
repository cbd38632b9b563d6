// Host side of the C ABI in include/pw_advect.h: plans, argument checks and
// kernel dispatch.  No entry point except pw_advect_plan allocates, and none
// synchronises.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "pw_advect.h"
#include "pw_kernels.hpp"
#include "pw_plan.hpp"

namespace {

thread_local int32_t g_last_hip_error = 0;

int32_t hip_fail(hipError_t e) {
    g_last_hip_error = static_cast<int32_t>(e);
    return PW_ERR_HIP;
}

}  // namespace

namespace pw {

int64_t elem_bytes(int32_t storage) {
    switch (storage) {
        case PW_F64: return 8;
        case PW_F32:
        case PW_I32: return 4;
        case PW_BF16:
        case PW_F16:
        case PW_I16: return 2;
        default: return 0;
    }
}

int64_t compute_bytes(int32_t storage) { return storage == PW_F64 || storage == PW_I32 ? 8 : 4; }

// The kernel height (template parameter NZ) of the march variant for a shape:
// its own, or minus its height class.
int32_t march_height(int32_t storage, const pw_shape& s) {
    return compiled_height(s.nz) && vector_shape(storage, s) ? s.nz : -kHeightClass[height_class(s.nz)];
}

// LDS of one march workgroup: three fields per ring slot (march_slots<CT>()).
int64_t march_lds_bytes(int32_t storage, int32_t chunk, int32_t height) {
    const int64_t slots = compute_bytes(storage) == 8 ? march_slots<double>() : march_slots<float>();
    return 3 * slots * march_wpad(chunk, height) * compute_bytes(storage);
}

bool scaled_storage(int32_t storage) {
    return storage == PW_BF16 || storage == PW_F16 || storage == PW_I16 || storage == PW_I32;
}

int32_t normalize_shape(const pw_shape& in, pw_shape* out) {
    pw_shape s = in;
    if (s.nx < 1 || s.ny < 1 || s.nz < 2 || s.reserved != 0) return PW_ERR_INVALID_ARG;
    const int64_t nx = s.nx, ny = s.ny, nz = s.nz;
    // 32-bit in-plane indexing in the kernels; plane indices up to nx + 1
    if ((ny + 2) * nz >= (int64_t(1) << 31) || nx + 2 >= (int64_t(1) << 31)) return PW_ERR_INVALID_ARG;
    // strides: every element offset stays below 2^48 (far beyond any device
    // memory), so element and byte offsets never overflow 64 bits
    constexpr int64_t kMaxElems = int64_t(1) << 48;
    if (s.sy == 0) s.sy = nz;
    if (s.sy < nz || s.sy > kMaxElems / (ny + 2)) return PW_ERR_INVALID_ARG;
    if (s.sx == 0) s.sx = (ny + 2) * s.sy;
    if (s.sx < (ny + 2) * s.sy || s.sx > kMaxElems / (nx + 2)) return PW_ERR_INVALID_ARG;
    *out = s;
    return PW_OK;
}

int64_t extent_elems(const pw_shape& s) {
    return (int64_t)(s.nz - 1) + ((int64_t)s.ny + 1) * s.sy + ((int64_t)s.nx + 1) * s.sx + 1;
}

bool march_possible(const pw_shape& s) {
    return s.sy == s.nz && s.nz <= kMarchMaxNz && s.nx <= (1 << 30);
}

// Even split of nx planes into segments of at most `seg`.
static int32_t even_seg(int32_t nx, int64_t seg) {
    seg = std::max<int64_t>(1, std::min<int64_t>(seg, nx));
    const int64_t n = (nx + seg - 1) / seg;
    return (int32_t)((nx + n - 1) / n);
}

// Planes per segment, from the tiles (segments x chunks) the split gives and
// the tiles the chip keeps resident (two workgroups per CU for FP64 compute,
// four for FP32 compute, fewer if the LDS holds fewer).
//
// 1. Whole rounds: on grids whose chunks divide evenly over the XCDs, about
//    8192 tiles (FP64, 16-bit types) or 2048 (4-byte types) of 16 .. 256
//    planes, if they fill whole rounds of resident tiles.  Tiles of equal
//    length then stay in step and meet each other's boundary planes and halo
//    columns in L2.  Measured over segments of 16 .. 256 planes: best on
//    2048 x 2048 x 64 for every type (64 planes for FP64, 256 for FP32) and
//    on 512 x 512 x 64 for FP64 (16 planes).
// 2. Otherwise, with `rounds` or more rounds of tiles: a split near the
//    type's best length `planes` (the more arithmetic and conversion per
//    byte, the more a tile's start costs and the longer the best segment).
// 3. Otherwise the split with the least predicted time: a tile of n planes
//    takes n + start plane steps; a full round of tiles is limited by the
//    HBM, and a step of a nearly empty chip still takes `idle` of a full
//    round's step (the latency of one plane); a started round costs `tail`
//    of what a full one does beyond its own tiles.
// Fitted to every even split of 58 random grids (16..2048 planes and rows,
// heights 64, 96, 128) for each type: 1.3% (FP64), 1.7% (FP32), 1.2% (16-bit
// types) and 0.8% (int32) behind the best split on average.  The first rule
// alone, for every grid, is 17-29% behind: it leaves small grids with too few
// tiles (64 x 64 x 64 FP64: 32 tiles, 16.9 us; 256 tiles, 5.9 us) and ragged
// ones with long tiles out of step (1100 x 1000 x 64 FP32: 2.07 rounds of 65
// planes, 387 us; 7.9 rounds of 17, 318 us).  The resident tiles are those of
// the compiled heights' kernels; the class kernels of FP32 and int32 for any
// height above 84 keep fewer (three and one per CU), and only FP64 has
// constants of its own for the classes, so their segments may be some percent
// off the best.
struct SegModel {
    int32_t planes;   // best segment length with many tiles
    double begin;     // a tile's start with many tiles, in plane steps
    double start;     // a tile's start with few tiles, in plane steps
    double idle, tail, rounds;
};

static int32_t model_seg(int32_t storage, const pw_shape& s, int32_t nchunks, int64_t lds_bytes) {
    constexpr int kCus = 256;
    // FP64 heights of a class: a longer best length (382 x 317 x 113: 20 planes
    // 138 us, 6 planes 151 us)
    constexpr SegModel f64{10, 0.0, 2.0, 0.4, 1.0, 3.0}, f64_class{14, 1.0, 2.0, 0.4, 1.0, 3.0}, f32{24, 0.0, 1.0, 0.4, 1.0, 3.0},
        w16{24, 1.0, 3.0, 0.3, 0.4, 3.0}, i32{64, 2.0, 2.0, 0.4, 0.4, 2.0};
    const SegModel& m = storage == PW_F64 ? (march_height(storage, s) < 0 ? f64_class : f64) : storage == PW_F32 ? f32 : storage == PW_I32 ? i32 : w16;
    const int64_t fit = std::max<int64_t>(1, kLdsPerCu / std::max<int64_t>(lds_bytes, 1));
    const double resident = (double)kCus * (double)std::min<int64_t>(compute_bytes(storage) == 8 ? 2 : 4, fit);
    auto segments = [&](int64_t n) { return ((int64_t)s.nx + n - 1) / n; };
    auto fill = [&](int64_t n) { return (double)nchunks * (double)segments(n) / resident; };

    const int64_t target = elem_bytes(storage) == 4 ? 2048 : 8192;
    const int32_t whole = even_seg(s.nx, std::min<int64_t>(std::max<int64_t>((int64_t)s.nx * nchunks / target, 16), 256));
    const double xw = fill(whole);
    if (nchunks % kNumXcd == 0 && xw >= 1.0 && std::ceil(xw) - xw < 0.05 * xw) return whole;

    auto rounds = [&](double x) { return x <= 1.0 ? m.idle + (1.0 - m.idle) * x : x + m.tail * (std::ceil(x) - x); };
    const int32_t near = even_seg(s.nx, ((int64_t)s.nx + segments(m.planes) - 1) / segments(m.planes));
    const bool many = fill(near) >= m.rounds;
    const double extra = many ? m.begin : m.start;
    const int64_t lo = many ? 2 * m.planes / 3 : 1, hi = std::min<int64_t>(2 * m.planes, s.nx);
    int32_t best = near;
    double low = (near + extra) * rounds(fill(near));
    for (int64_t n = lo; n <= hi; ++n) {
        if (even_seg(s.nx, n) != n) continue;   // an even split of its own
        const double t = ((double)n + extra) * rounds(fill(n));
        if (t < low) {
            low = t;
            best = (int32_t)n;
        }
    }
    return best;
}

// The model's segments, longer where they are more than a launch may hold.
int32_t auto_seg(int32_t storage, const pw_shape& s, int32_t nchunks, int64_t lds_bytes) {
    int32_t seg = model_seg(storage, s, nchunks, lds_bytes);
    while ((int64_t)nchunks * (((int64_t)s.nx + seg - 1) / seg) > kMaxTiles) seg = even_seg(s.nx, 2 * (int64_t)seg);
    return seg;
}

// Default workgroup and planes per segment of the direct variant.  A wave
// carries its planes from step to step, so segments only have to be long
// enough to spread the two extra planes of their start, and short ones keep
// neighbouring waves within reach of each other's rows in L1 and L2: 4 planes
// for FP64 compute and 8 for FP32 compute are best or within 4% of the best
// of 1, 2, 4, 8, 16, 32 on grids from 5 to 74 million points (250 x 310 x 60
// padded FP64: 58 us with 4, 64 with 8, 77 with 1; 500 x 500 x 199 padded
// BF16: 230 with 8, 234 with 4, 390 with 1), 2 on grids that do not fill the
// chip (kWaves waves in flight).  Large grids take workgroups of 512 threads,
// whose eight waves share more rows: FP64 from 4 million points on (250 x 310 x
// 60 padded 58 against 61 us, 512 x 512 x 64 181 against 195), int32 and the
// 16-bit types from 16 million on (500 x 500 x 199 padded int32 388 against
// 421 us, BF16 230 against 246; 250 x 310 x 60 int32 32 against 29, hence the
// line); FP32 is indifferent (404 against 400 us) and keeps 256.
static int32_t direct_block(int32_t storage, const pw_shape& s) {
    const int64_t pairs = (int64_t)s.ny * (((int64_t)s.nz + 1) / 2) * s.nx;
    if (storage == PW_F32) return 256;
    return pairs >= (int64_t(1) << (storage == PW_F64 ? 21 : 23)) ? 512 : 256;
}
static int32_t direct_seg(int32_t storage, const pw_shape& s, int32_t nchunks, int32_t block) {
    constexpr int64_t kWaves = 256 * 12;
    const int64_t most = compute_bytes(storage) == 8 ? 4 : 8;
    int64_t seg = (int64_t)nchunks * (block / 64) * s.nx / kWaves;
    seg = std::max<int64_t>(2, std::min<int64_t>(seg, most));
    // the grid's limit: fewer than 2^32 threads
    while (seg < s.nx && (int64_t)nchunks * ((s.nx + seg - 1) / seg) * block >= (int64_t(1) << 32)) seg *= 2;
    return even_seg(s.nx, seg);
}

int32_t resolve_launch(int32_t storage, const pw_shape& s, const pw_tuning& t, Launch* L) {
    Launch r{};
    int32_t variant = t.variant;
    if (variant == PW_VARIANT_AUTO) variant = march_possible(s) ? PW_VARIANT_MARCH : PW_VARIANT_DIRECT;
    if (variant != PW_VARIANT_MARCH && variant != PW_VARIANT_DIRECT) return PW_ERR_UNSUPPORTED;
    if (variant == PW_VARIANT_MARCH && !march_possible(s)) return PW_ERR_UNSUPPORTED;
    r.variant = variant;
    if (variant == PW_VARIANT_MARCH) {
        const int32_t chunk = t.chunk ? t.chunk : 512;
        if (chunk != 256 && chunk != 512 && chunk != 1024) return PW_ERR_INVALID_ARG;
        if (t.seg < 0) return PW_ERR_INVALID_ARG;
        r.chunk = chunk;
        r.block = 256;
        r.nchunks = (int32_t)(((int64_t)s.ny * s.nz + chunk - 1) / chunk);
        r.lds_bytes = march_lds_bytes(storage, chunk, march_height(storage, s));
        if (r.lds_bytes > kMaxDynamicLds) return PW_ERR_UNSUPPORTED;
        r.seg = t.seg ? std::min(t.seg, s.nx) : auto_seg(storage, s, r.nchunks, r.lds_bytes);
        r.nseg = (s.nx + r.seg - 1) / r.seg;
    } else {
        const int32_t block = t.block ? t.block : direct_block(storage, s);
        if (block != 64 && block != 128 && block != 256 && block != 512) return PW_ERR_INVALID_ARG;
        if (s.nx > 65535) return PW_ERR_INVALID_ARG;
        r.block = block;
        r.chunk = 0;
        const int64_t pairs = s.ny * (((int64_t)s.nz + 1) / 2);   // a lane takes two levels
        const int64_t per = block / 64 * kDirectPairs;
        r.nchunks = (int32_t)((pairs + per - 1) / per);
        r.lds_bytes = 0;
        r.seg = direct_seg(storage, s, r.nchunks, block);
        r.nseg = (s.nx + r.seg - 1) / r.seg;
    }
    r.tiles = (int64_t)r.nchunks * r.nseg;
    // compact tile order (march_compact_tile) when every XCD owns a chunk
    r.run = r.nchunks >= kNumXcd ? march_run(r.nchunks) : 0;
    r.blocks = r.run > 0 ? (int32_t)(r.tiles / (kNumXcd * r.run)) : 0;
    const int64_t rem = r.tiles - (int64_t)r.blocks * kNumXcd * r.run;
    r.workgroups = r.run > 0 ? kNumXcd * ((int64_t)r.blocks * r.run + (rem + kNumXcd - 1) / kNumXcd) : r.tiles;
    if (r.workgroups >= (int64_t(1) << 31)) return PW_ERR_INVALID_ARG;
    *L = r;
    return PW_OK;
}

// ---------------------------------------------------------------------------
// launches
// ---------------------------------------------------------------------------
template <typename ST, int P, int NZ, bool EVEN>
hipError_t launch_march(const DomainArgs& d, const Launch& L, hipStream_t stream) {
    auto kern = pw_march_kernel<ST, 256, P, NZ, EVEN>;
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [&] {
        attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kMaxDynamicLds);
    });
    if (attr_err != hipSuccess) return attr_err;
    MarchGeom g{L.nchunks, L.nseg, L.seg, L.run, L.blocks};
    using CT = typename compute_of<ST>::type;
    const size_t lds = 3 * sizeof(CT) * march_slots<CT>() * march_wpad(P, NZ);
    hipLaunchKernelGGL(kern, dim3((unsigned)L.workgroups), dim3(256), lds, stream, d, g);
    return hipGetLastError();
}

template <typename ST, int NZ, bool EVEN>
hipError_t dispatch_march_p(const DomainArgs& d, const Launch& L, hipStream_t stream) {
    switch (L.chunk) {
        case 256: return launch_march<ST, 256, NZ, EVEN>(d, L, stream);
        case 512: return launch_march<ST, 512, NZ, EVEN>(d, L, stream);
        case 1024: return launch_march<ST, 1024, NZ, EVEN>(d, L, stream);
        default: return hipErrorInvalidValue;
    }
}

template <typename ST>
hipError_t launch_direct(const DomainArgs& d, const Launch& L, hipStream_t stream) {
    const MarchGeom g{L.nchunks, L.nseg, L.seg, L.run, L.blocks};
    const dim3 grid((unsigned)L.workgroups), block((unsigned)L.block);
    const bool narrow = ((int64_t)d.ny + 2) * d.sy * (int64_t)sizeof(ST) < (int64_t(1) << 31);
    if (!narrow) hipLaunchKernelGGL((pw_direct_kernel<ST, int64_t, true>), grid, block, 0, stream, d, g);
    else if (d.nz % 2) hipLaunchKernelGGL((pw_direct_kernel<ST, uint32_t, true>), grid, block, 0, stream, d, g);
    else hipLaunchKernelGGL((pw_direct_kernel<ST, uint32_t, false>), grid, block, 0, stream, d, g);
    return hipGetLastError();
}

template <typename ST, bool EVEN>
hipError_t launch_class(const DomainArgs& d, const Launch& L, hipStream_t stream) {
    switch (height_class(d.nz)) {
        case 0: return dispatch_march_p<ST, -kHeightClass[0], EVEN>(d, L, stream);
        case 1: return dispatch_march_p<ST, -kHeightClass[1], EVEN>(d, L, stream);
        default: return dispatch_march_p<ST, -kHeightClass[2], EVEN>(d, L, stream);
    }
}

template <typename ST>
hipError_t launch_typed(const DomainArgs& d, const Launch& L, bool vec, hipStream_t stream) {
    // Column heights 64 (the paper's and MONC's default), 96 and 128 get
    // kernels with the height compiled in where every vector is aligned;
    // other heights and alignments use the kernel of their height class,
    // whose windows are moved in whole vectors and whose threads take pairs of
    // points too.  Against the kernel they had before (one point per thread,
    // every LDS address computed, element loads for odd heights or
    // alignments): 300 x 420 x 80 FP64 131 -> 93 us (5.2 TB/s algorithmic),
    // 257 x 391 x 63 FP32 57 -> 34 us (4.4 TB/s), 160 x 180 x 165 BF16
    // 59 -> 24 us.  Even heights have kernels of their own, whose LDS reads
    // are aligned pairs (300 x 420 x 80 FP64 101 -> 93 us, BF16 38 -> 29 us
    // against the kernel for any height, whose 4-byte reads at an 8-byte
    // stride conflict in the banks).
    if (L.variant == PW_VARIANT_MARCH) {
        if (vec) {
            switch (d.nz) {
                case 64: return dispatch_march_p<ST, 64, true>(d, L, stream);
                case 96: return dispatch_march_p<ST, 96, true>(d, L, stream);
                case 128: return dispatch_march_p<ST, 128, true>(d, L, stream);
                default: break;
            }
        }
        return d.nz % 2 == 0 ? launch_class<ST, true>(d, L, stream) : launch_class<ST, false>(d, L, stream);
    }
    return launch_direct<ST>(d, L, stream);
}

hipError_t launch_domain(int32_t storage, const DomainArgs& d, const Launch& L, bool vec, hipStream_t stream) {
    switch (storage) {
        case PW_F64: return launch_typed<double>(d, L, vec, stream);
        case PW_F32: return launch_typed<float>(d, L, vec, stream);
        case PW_BF16: return launch_typed<bf16_t>(d, L, vec, stream);
        case PW_F16: return launch_typed<f16_t>(d, L, vec, stream);
        case PW_I16: return launch_typed<fx16_t>(d, L, vec, stream);
        case PW_I32: return launch_typed<fx32_t>(d, L, vec, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace pw

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------
using namespace pw;

extern "C" {

const char* pw_status_string(int32_t status) {
    switch (status) {
        case PW_OK: return "ok";
        case PW_ERR_INVALID_ARG: return "invalid argument";
        case PW_ERR_UNSUPPORTED: return "unsupported";
        case PW_ERR_ALIAS: return "an output overlaps an input or another output";
        case PW_ERR_ALIGNMENT: return "misaligned pointer";
        case PW_ERR_OUT_OF_MEMORY: return "out of device memory";
        case PW_ERR_HIP: return "HIP runtime error";
        case PW_ERR_CAPTURE: return "allocation requested during stream capture";
        case PW_ERR_PLAN_MISMATCH: return "arguments do not match the plan";
        default: return "unknown status";
    }
}

int32_t pw_last_hip_error(void) { return g_last_hip_error; }

int32_t pw_advect_plan(pw_plan** plan, int32_t storage, const pw_shape* shapes, int32_t ndomains,
                       const pw_tuning* tuning) {
    if (!plan || !shapes || ndomains < 1) return PW_ERR_INVALID_ARG;
    *plan = nullptr;
    if (elem_bytes(storage) == 0) return PW_ERR_UNSUPPORTED;
    pw_tuning t{};
    if (tuning) t = *tuning;
    std::unique_ptr<pw_plan> p(new (std::nothrow) pw_plan());
    if (!p) return PW_ERR_OUT_OF_MEMORY;
    p->storage = storage;
    p->ndomains = ndomains;
    p->tuning = t;
    p->shapes.resize(ndomains);
    for (int32_t d = 0; d < ndomains; ++d) {
        int32_t rc = normalize_shape(shapes[d], &p->shapes[d]);
        if (rc != PW_OK) return rc;
        p->points += (int64_t)p->shapes[d].nx * p->shapes[d].ny * p->shapes[d].nz;
    }
    if (ndomains == 1) {
        int32_t rc = resolve_launch(storage, p->shapes[0], t, &p->single);
        if (rc != PW_OK) return rc;
    }
    int32_t rc = batched_plan_init(p.get());
    if (rc != PW_OK) return rc;
    *plan = p.release();
    return PW_OK;
}

int32_t pw_plan_destroy(pw_plan* plan) {
    if (!plan) return PW_OK;
    int32_t rc = batched_plan_free(plan);
    delete plan;
    return rc;
}

int32_t pw_plan_get_info(const pw_plan* plan, pw_plan_info* info) {
    if (!plan || !info) return PW_ERR_INVALID_ARG;
    pw_plan_info r{};
    r.storage = plan->storage;
    r.ndomains = plan->ndomains;
    const Launch& L = plan->ndomains == 1 ? plan->single : plan->batch.launch;
    if (plan->ndomains == 1) {
        r.batched_workgroups = plan->batch.launch.workgroups;
    } else {
        r.batched_workgroups = L.workgroups;
    }
    r.variant = L.variant;
    r.chunk = L.chunk;
    r.seg = L.seg;
    r.block = L.block;
    r.workgroups = L.workgroups;
    r.tiles = L.tiles;
    r.lds_bytes = L.lds_bytes;
    r.points = plan->points;
    *info = r;
    return PW_OK;
}

int32_t pw_advect(const pw_plan* plan, const void* u, const void* v, const void* w, void* su, void* sv,
                  void* sw, double tcx, double tcy, const double* tzc1, const double* tzc2,
                  const double* tzd1, const double* tzd2, const pw_scales* scales, void* stream) {
    if (!plan) return PW_ERR_INVALID_ARG;
    if (plan->ndomains != 1) return PW_ERR_PLAN_MISMATCH;
    if (!u || !v || !w || !su || !sv || !sw || !tzc1 || !tzc2 || !tzd1 || !tzd2) return PW_ERR_INVALID_ARG;
    if (!std::isfinite(tcx) || !std::isfinite(tcy)) return PW_ERR_INVALID_ARG;
    const pw_shape& s = plan->shapes[0];
    const int64_t eb = elem_bytes(plan->storage);

    const void* ins[3] = {u, v, w};
    void* outs[3] = {su, sv, sw};
    for (const void* q : ins)
        if (reinterpret_cast<uintptr_t>(q) % eb) return PW_ERR_ALIGNMENT;
    for (const void* q : outs)
        if (reinterpret_cast<uintptr_t>(q) % eb) return PW_ERR_ALIGNMENT;
    for (const double* q : {tzc1, tzc2, tzd1, tzd2})
        if (reinterpret_cast<uintptr_t>(q) % 8) return PW_ERR_ALIGNMENT;
    const int64_t ext = extent_elems(s) * eb;
    if (any_overlap(ins, outs, ext)) return PW_ERR_ALIAS;

    DomainArgs d{};
    int32_t rc = fill_domain_args(plan->storage, s, u, v, w, su, sv, sw, tcx, tcy, tzc1, tzc2, tzd1, tzd2,
                                  scales, &d);
    if (rc != PW_OK) return rc;
    const bool vec = vector_ok(plan->storage, s, ins, outs);
    hipError_t e = launch_domain(plan->storage, d, plan->single, vec, static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return hip_fail(e);
    return PW_OK;
}

}  // extern "C"

namespace pw {

int32_t report_hip(hipError_t e) { return hip_fail(e); }

bool any_overlap(const void* const ins[3], void* const outs[3], int64_t ext) {
    auto lo = [](const void* q) { return reinterpret_cast<uintptr_t>(q); };
    for (int a = 0; a < 3; ++a) {
        const uintptr_t oa = lo(outs[a]);
        for (int b = 0; b < 3; ++b) {
            const uintptr_t ib = lo(ins[b]);
            if (oa < ib + ext && ib < oa + ext) return true;
        }
        for (int b = a + 1; b < 3; ++b) {
            const uintptr_t ob = lo(outs[b]);
            if (oa < ob + ext && ob < oa + ext) return true;
        }
    }
    return false;
}

bool vector_shape(int32_t storage, const pw_shape& s) {
    const int64_t vw = 16 / elem_bytes(storage);
    return s.nz % vw == 0 && s.sx % vw == 0 && s.sy % vw == 0;
}

bool vector_ok(int32_t storage, const pw_shape& s, const void* const ins[3], void* const outs[3]) {
    if (!vector_shape(storage, s)) return false;
    for (int a = 0; a < 3; ++a) {
        if (reinterpret_cast<uintptr_t>(ins[a]) % 16 || reinterpret_cast<uintptr_t>(outs[a]) % 16) return false;
    }
    return true;
}

int32_t fill_domain_args(int32_t storage, const pw_shape& s, const void* u, const void* v, const void* w,
                         void* su, void* sv, void* sw, double tcx, double tcy, const double* tzc1,
                         const double* tzc2, const double* tzd1, const double* tzd2, const pw_scales* scales,
                         DomainArgs* out) {
    DomainArgs d{};
    d.u = u;
    d.v = v;
    d.w = w;
    d.su = su;
    d.sv = sv;
    d.sw = sw;
    d.tzc1 = tzc1;
    d.tzc2 = tzc2;
    d.tzd1 = tzd1;
    d.tzd2 = tzd2;
    float in_s[3] = {1.0f, 1.0f, 1.0f};
    float out_s[3] = {1.0f, 1.0f, 1.0f};
    if (scales && scaled_storage(storage)) {
        for (int f = 0; f < 3; ++f) {
            const float a = scales->in_scale[f];
            const float b = scales->out_scale[f];
            if (!(a > 0.0f) || !std::isfinite(a) || !(b > 0.0f) || !std::isfinite(b)) return PW_ERR_INVALID_ARG;
            int ea, eb;
            if (std::frexp(a, &ea) != 0.5f || std::frexp(b, &eb) != 0.5f) return PW_ERR_INVALID_ARG;
            in_s[f] = a;
            out_s[f] = b;
        }
    }
    fold_coefficients(tcx, tcy, in_s, out_s, d.cx, d.cy, d.cz);
    d.nx = s.nx;
    d.ny = s.ny;
    d.nz = s.nz;
    d.sy = s.sy;
    d.sx = s.sx;
    *out = d;
    return PW_OK;
}

}  // namespace pw
