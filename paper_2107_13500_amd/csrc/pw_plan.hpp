// Internal plan layout and host helpers shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <memory>
#include <vector>

#include "pw_advect.h"
#include "pw_kernels.hpp"

namespace pw {

// Resolved launch shape of one domain (or of the batched kernel).
struct Launch {
    int32_t variant = 0;
    int32_t chunk = 0;     // march: points per workgroup chunk
    int32_t seg = 0;       // planes per segment
    int32_t block = 0;     // threads per workgroup
    int32_t nchunks = 0;   // chunks per plane (direct: workgroups' shares of its pairs)
    int32_t nseg = 0;      // segments
    int32_t run = 0;       // compact tile order, neighbouring tiles per XCD and block (0: not used)
    int32_t blocks = 0;    // compact tile order, full blocks of tiles
    int64_t workgroups = 0;
    int64_t tiles = 0;
    int64_t lds_bytes = 0;
};

// Device table of a batched plan (one entry per domain).
struct BatchDomain {
    int32_t nx, ny, nz;
    int32_t nchunks;
    int32_t nseg;
    int32_t seg;          // planes per segment: nx split into nseg even parts
    int64_t sy, sx;
    int64_t tile_begin;   // first global tile of this domain
    int32_t rec;          // index of the domain's record in the caller's pw_domain_args array
    int32_t fill_begin;   // first workgroup of this domain in the perturbation's own split
};

struct BatchState {
    Launch launch;               // shared kernel shape (chunk, bound of the segments, LDS)
    BatchDomain* d_table = nullptr;
    unsigned long long* d_errors = nullptr;
    const int32_t* d_order = nullptr;   // one workgroup per tile: each workgroup's tile (-1: none), or NULL
    int device = -1;
    int32_t fill_planes = 0;     // the perturbation's split: most planes of a workgroup,
    int64_t fill_tiles = 0;      // and its workgroups (0: more than one launch may hold)
    bool vec_shapes = false;     // every shape allows 16-byte loads
    int32_t kind = 0;            // code paths of the batched kernel (BatchKind in pw_batched.hip)
};

}  // namespace pw

struct pw_plan {
    int32_t storage = 0;
    int32_t ndomains = 0;
    pw_tuning tuning{};
    std::vector<pw_shape> shapes;   // strides normalised
    int64_t points = 0;
    pw::Launch single;              // ndomains == 1
    pw::BatchState batch;           // ndomains >= 1 (batched entry point)
};

namespace pw {

int64_t elem_bytes(int32_t storage);
int64_t compute_bytes(int32_t storage);
int32_t march_height(int32_t storage, const pw_shape& s);
int64_t march_lds_bytes(int32_t storage, int32_t chunk, int32_t height);
bool scaled_storage(int32_t storage);   // 16-bit and int32 types: per-field scales
int32_t normalize_shape(const pw_shape& in, pw_shape* out);
int64_t extent_elems(const pw_shape& s);
bool march_possible(const pw_shape& s);
int32_t auto_seg(int32_t storage, const pw_shape& s, int32_t nchunks, int64_t lds_bytes);
int32_t resolve_launch(int32_t storage, const pw_shape& s, const pw_tuning& t, Launch* L);
bool any_overlap(const void* const ins[3], void* const outs[3], int64_t ext);
bool vector_shape(int32_t storage, const pw_shape& s);   // every vector of 16-byte aligned arrays is aligned
bool vector_ok(int32_t storage, const pw_shape& s, const void* const ins[3], void* const outs[3]);
int32_t fill_domain_args(int32_t storage, const pw_shape& s, const void* u, const void* v, const void* w,
                         void* su, void* sv, void* sw, double tcx, double tcy, const double* tzc1,
                         const double* tzc2, const double* tzd1, const double* tzd2, const pw_scales* scales,
                         DomainArgs* out);
int32_t report_hip(hipError_t e);

// batched plans (pw_batched.hip)
int32_t batched_plan_init(pw_plan* p);
int32_t batched_plan_free(pw_plan* p);
int32_t record_timestep(const pw_plan* plan, const pw_domain_args* d_args, uint64_t seed, unsigned long long* d_call,
                        double amplitude, hipStream_t s);

}  // namespace pw
