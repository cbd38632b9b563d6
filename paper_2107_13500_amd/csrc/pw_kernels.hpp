// PW advection kernels for gfx950.
//
// direct  one lane per pair of levels, walking along x; every operand is a
//         global load or a neighbouring lane's, the reuse of the rows j-1 and
//         j+1 is left to L1/L2.  Handles any strides and heights.
// march   the HBM-streaming kernel.  With packed columns (sy = nz) each x plane
//         is one contiguous run of (ny + 2) * nz elements, so a workgroup owns a
//         contiguous chunk of P points of that (j, k) run and walks along x.  It
//         keeps the planes i-1, i, i+1 of u, v, w in a ring of LDS slots (the
//         GPU form of the paper's three-slice shift buffer, Sec. III; a fourth
//         slot for FP32 compute saves one barrier per plane).  The window of a
//         plane is [p0 - nz, p0 + P + nz) -- the chunk plus one column of y
//         halo on each side -- so every input element crosses HBM about once.
//         Two or three later planes are in flight in registers while a plane
//         is computed.  The ring rotation is unrolled so slots and register
//         sets are compile-time, and each thread computes two consecutive
//         points, sharing their neighbour reads and storing both results with
//         one vector store.  With a compile-time column height every LDS
//         offset is an immediate; for other heights the window's LDS pitch is
//         that of a height class, so only the three rows j-1, j, j+1 need a
//         base address of their own.
#pragma once

#include <type_traits>

#include "pw_stencil.hpp"
#include "pw_tiles.hpp"

namespace pw {

constexpr int kMarchMaxNz = 256;   // largest column the march variant accepts
// Height classes of the march kernel for column heights without a kernel of
// their own: the kernel of class H stages windows of up to P + 2 H elements.
// The bounds are where one more load round per thread begins at P = 512 (84:
// two rounds of 4-element vectors for FP32 compute, four of 2-element ones for
// FP64 compute; 170: five for FP64 compute, and the largest window with four
// FP32-compute workgroups per CU in LDS).
constexpr int kHeightClass[3] = {84, 170, kMarchMaxNz};
__host__ __device__ constexpr int height_class(int nz) { return nz <= kHeightClass[0] ? 0 : (nz <= kHeightClass[1] ? 1 : 2); }
constexpr bool compiled_height(int nz) { return nz == 64 || nz == 96 || nz == 128; }
constexpr int kLdsPerCu = 160 * 1024;           // gfx950 LDS per CU (and per workgroup)
constexpr int kMaxDynamicLds = kLdsPerCu - 1024;   // leaves room for a kernel's small static LDS
// A launch holds fewer than 2^32 threads: workgroups of 256, a block of 64 of
// them left for the padding of the tile orders.
constexpr int64_t kMaxTiles = (int64_t(1) << 24) - 64;
constexpr int kNumXcd = 8;         // MI355X: 8 accelerator complex dies, one L2 each

// Everything a kernel needs about one domain (passed by value).
struct DomainArgs {
    const void* u;
    const void* v;
    const void* w;
    void* su;
    void* sv;
    void* sw;
    const double* tzc1;
    const double* tzc2;
    const double* tzd1;
    const double* tzd2;
    // Per output (su, sv, sw): x and y coefficients and the factor applied to
    // the per-level vertical coefficients, with the storage scales of 16-bit
    // and int32 storage folded in (all exact powers of two); plain tcx, tcy,
    // 1 otherwise.
    double cx[3], cy[3], cz[3];
    int32_t nx, ny, nz;
    int32_t pad_;
    int64_t sy, sx;
};

// Geometry of a march launch over one domain.
struct MarchGeom {
    int32_t nchunks;   // chunks of P points over the interior (j, k) run
    int32_t nseg;      // x segments
    int32_t seg;       // planes per segment
    int32_t run;       // compact tile order: neighbouring tiles per XCD and block (0: XCD-contiguous order)
    int32_t blocks;    // compact tile order: full blocks of kNumXcd * run tiles
};

// Storage types that carry per-field power-of-two scales.
template <typename ST> struct scaled_type { static constexpr bool value = false; };
template <> struct scaled_type<bf16_t> { static constexpr bool value = true; };
template <> struct scaled_type<f16_t> { static constexpr bool value = true; };
template <> struct scaled_type<fx16_t> { static constexpr bool value = true; };
template <> struct scaled_type<fx32_t> { static constexpr bool value = true; };

// Folded coefficients (see DomainArgs) from tcx, tcy and the storage scales.
__host__ __device__ inline void fold_coefficients(double tcx, double tcy, const float in_scale[3],
                                                  const float out_scale[3], double cx[3], double cy[3],
                                                  double cz[3]) {
    const double su = in_scale[0], sv = in_scale[1], sw = in_scale[2];
    const double o[3] = {out_scale[0], out_scale[1], out_scale[2]};
    const double own[3] = {su, sv, sw};
    for (int f = 0; f < 3; ++f) {
        cx[f] = tcx * o[f] / (own[f] * su);
        cy[f] = tcy * o[f] / (own[f] * sv);
        cz[f] = o[f] / (own[f] * sw);
    }
}

// Vectors of N elements of type T that are only aligned to A bytes.
template <typename T, int N, int A> struct vec_at;
#define PW_VEC_AT(T, N, A) \
    template <> struct vec_at<T, N, A> { typedef T type __attribute__((ext_vector_type(N), aligned(A))); };
PW_VEC_AT(uint32_t, 4, 4)
PW_VEC_AT(uint32_t, 4, 8)
PW_VEC_AT(uint32_t, 4, 16)
PW_VEC_AT(uint32_t, 2, 2)
PW_VEC_AT(uint32_t, 2, 4)
PW_VEC_AT(uint32_t, 2, 8)
PW_VEC_AT(uint32_t, 1, 2)
PW_VEC_AT(uint32_t, 1, 4)
PW_VEC_AT(int32_t, 2, 4)
PW_VEC_AT(int32_t, 2, 8)
PW_VEC_AT(float, 2, 4)
PW_VEC_AT(float, 2, 8)
PW_VEC_AT(double, 2, 8)
PW_VEC_AT(double, 2, 16)
#undef PW_VEC_AT

// One load of a Raw value (8 or 16 bytes, aligned to ALIGN bytes) through a
// global pointer, as a plain integer vector (HIP's vector structs cannot be
// assigned from an address-space-qualified lvalue), copied bit for bit.
template <typename Raw, int ALIGN>
__device__ __forceinline__ Raw load_global(global_ptr<const char> p) {
    static_assert(sizeof(Raw) == 8 || sizeof(Raw) == 16, "8 or 16 bytes");
    using V = typename vec_at<uint32_t, sizeof(Raw) / 4, ALIGN>::type;
    const V x = *reinterpret_cast<global_ptr<const V>>(p);
    Raw r;
    __builtin_memcpy(&r, &x, sizeof(Raw));
    return r;
}

template <typename ST>
__device__ __forceinline__ void store_out(global_ptr<ST> p, typename compute_of<ST>::type x) {
    ST y = from_compute<ST>(x);
    if constexpr (sizeof(ST) == 2) {
        uint16_t bits;
        __builtin_memcpy(&bits, &y, 2);
        __builtin_nontemporal_store(bits, reinterpret_cast<global_ptr<uint16_t>>(p));
    } else if constexpr (std::is_same<ST, fx32_t>::value) {
        __builtin_nontemporal_store(y.v, reinterpret_cast<global_ptr<int32_t>>(p));
    } else {
        __builtin_nontemporal_store(y, p);
    }
}

// Two consecutive outputs p[0], p[1] with one store (p aligned to ALIGN elements).
// BF16 and FP16 pairs are rounded by one packed conversion (v_cvt_pk_bf16_f32,
// v_cvt_pk_f16_f32: round to nearest even, as from_compute).
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
template <typename ST, int ALIGN>
__device__ __forceinline__ void store_pair(global_ptr<ST> p, typename compute_of<ST>::type a, typename compute_of<ST>::type b) {
    constexpr int A = ALIGN * (int)sizeof(ST);
    if constexpr (std::is_same<ST, double>::value) {
        using f64x2a = typename vec_at<double, 2, A>::type;
        __builtin_nontemporal_store(f64x2a{a, b}, reinterpret_cast<global_ptr<f64x2a>>(p));
    } else if constexpr (std::is_same<ST, float>::value) {
        using f32x2a = typename vec_at<float, 2, A>::type;
        __builtin_nontemporal_store(f32x2a{a, b}, reinterpret_cast<global_ptr<f32x2a>>(p));
    } else if constexpr (std::is_same<ST, fx32_t>::value) {
        using i32x2 = typename vec_at<int32_t, 2, A>::type;
        __builtin_nontemporal_store(i32x2{from_compute<ST>(a).v, from_compute<ST>(b).v}, reinterpret_cast<global_ptr<i32x2>>(p));
    } else if constexpr (std::is_same<ST, bf16_t>::value || std::is_same<ST, f16_t>::value) {
        using H2 = typename std::conditional<std::is_same<ST, bf16_t>::value, bf16x2, f16x2>::type;
        const H2 h = __builtin_convertvector(f32x2{a, b}, H2);
        uint32_t bits;
        __builtin_memcpy(&bits, &h, 4);
        using u32a = typename vec_at<uint32_t, 1, A>::type;
        __builtin_nontemporal_store(u32a(bits), reinterpret_cast<global_ptr<u32a>>(p));
    } else {
        // int16, the result of from_compute in fewer instructions: clamp to
        // the int16 range (NaN becomes -32768), then add 1.5 * 2^23.  The sum
        // lies in [2^23, 2^24), where FP32 values are the integers, so the
        // addition itself rounds to the nearest integer, ties to even (the
        // offset is even); the offset is a multiple of 2^16, so the low 16
        // bits of the sum are that integer in two's complement.  One byte
        // permutation packs the two low halves.  (Clamping before rounding
        // gives the same result: the bounds are integers.)
        static_assert(std::is_same<ST, fx16_t>::value, "int16 fixed point");
        constexpr float kRoundOffset = 12582912.0f;   // 1.5 * 2^23
        const float ra = __builtin_fminf(__builtin_fmaxf(a, -32768.0f), 32767.0f) + kRoundOffset;
        const float rb = __builtin_fminf(__builtin_fmaxf(b, -32768.0f), 32767.0f) + kRoundOffset;
        // bytes 0, 1 of ra, then bytes 0, 1 of rb
        const uint32_t bits = __builtin_amdgcn_perm(__float_as_uint(rb), __float_as_uint(ra), 0x05040100u);
        using u32a = typename vec_at<uint32_t, 1, A>::type;
        __builtin_nontemporal_store(u32a(bits), reinterpret_cast<global_ptr<u32a>>(p));
    }
}

template <typename ST>
__device__ __forceinline__ PointCoefs<typename compute_of<ST>::type> point_coefs(const DomainArgs& d, int k) {
    using CT = typename compute_of<ST>::type;
    PointCoefs<CT> c;
    c.xu = static_cast<CT>(d.cx[0]);
    c.yu = static_cast<CT>(d.cy[0]);
    c.xv = static_cast<CT>(d.cx[1]);
    c.yv = static_cast<CT>(d.cy[1]);
    c.xw = static_cast<CT>(d.cx[2]);
    c.yw = static_cast<CT>(d.cy[2]);
    double z1 = 0.0, z2 = 0.0, e1 = 0.0, e2 = 0.0;
    if (k >= 2) {
        z1 = as_global(d.tzc1)[k - 1];
        z2 = as_global(d.tzc2)[k - 1];
        if (k < d.nz) {
            e1 = as_global(d.tzd1)[k - 1];
            e2 = as_global(d.tzd2)[k - 1];
        }
    }
    c.z1u = static_cast<CT>(z1 * d.cz[0]);
    c.z2u = static_cast<CT>(z2 * d.cz[0]);
    c.z1v = static_cast<CT>(z1 * d.cz[1]);
    c.z2v = static_cast<CT>(z2 * d.cz[1]);
    c.z1w = static_cast<CT>(e1 * d.cz[2]);
    c.z2w = static_cast<CT>(e2 * d.cz[2]);
    return c;
}

// ---------------------------------------------------------------------------
// march variant
// ---------------------------------------------------------------------------

// Workgroups are dispatched round-robin over the XCDs (workgroup b runs on
// XCD b mod 8), in order of b.  Two tile orders follow from that; both take
// the tiles from the chunk-fastest list (tile = segment * nchunks + chunk).
//
// Compact order (march_compact_tile), used when a plane has at least 8
// chunks: the list is cut into blocks of 8 R tiles, R about nchunks / 8
// (march_run), and XCD x takes run x of every block, so at any time all XCDs
// work on the same one or two segments -- the HBM traffic of the whole chip
// stays in a narrow band of x planes -- while the R chunks of a run share
// their y-halo columns in one XCD's L2.  The tiles past the last full block
// are split evenly too, so no XCD has more than one tile above the mean
// whatever nchunks is.  Measured on 2048 x 2048 x 64 against the
// XCD-contiguous order: FP64 3-4% faster, BF16 2-3%; on 512 x 512 x 64 FP64
// with 16-plane segments 14% faster.
//
// XCD-contiguous order (xcd_tile), for fewer than 8 chunks per plane: each
// XCD receives a contiguous range of the chunk-fastest tile list.
__host__ __device__ inline int march_run(int nchunks) { return (nchunks + kNumXcd / 2) / kNumXcd; }
// Tile of workgroup b, or -1 (no tile: b lies in the padding of the last block).
__host__ __device__ inline int march_compact_tile(int b, int ntiles, int run, int blocks) {
    const int x = b % kNumXcd;
    const int slot = b / kNumXcd;
    const int full = blocks * run;   // slots of each XCD in the full blocks
    if (slot < full) return ((slot / run) * kNumXcd + x) * run + slot % run;
    const int first = full * kNumXcd;
    const int rem = ntiles - first;   // < 8 run
    const int t = x * rem / kNumXcd + slot - full;
    return t < (x + 1) * rem / kNumXcd ? first + t : -1;
}
__device__ __forceinline__ int xcd_tile(int b, int G) {
    const int q = G / kNumXcd;
    const int r = G % kNumXcd;
    const int x = b % kNumXcd;
    const int slot = b / kNumXcd;
    return x * q + (x < r ? x : r) + slot;
}

// LDS reads around one point; NZ > 0 makes every offset an immediate.
template <typename CT, int NZ, int WPAD>
struct LdsAcc {
    const CT* m;   // plane i-1 at the point's window index
    const CT* c;   // plane i
    const CT* p;   // plane i+1
    int nz_rt;
    __device__ __forceinline__ int nz() const { return NZ > 0 ? NZ : nz_rt; }
    __device__ __forceinline__ static constexpr int wp() { return WPAD; }
    template <int di> __device__ __forceinline__ const CT* sel() const {
        return di < 0 ? m : (di > 0 ? p : c);
    }
    template <int dk, int dj, int di>
    __device__ __forceinline__ CT u() const { return sel<di>()[dk + dj * nz()]; }
    template <int dk, int dj, int di>
    __device__ __forceinline__ CT v() const { return sel<di>()[wp() + dk + dj * nz()]; }
    template <int dk, int dj, int di>
    __device__ __forceinline__ CT w() const { return sel<di>()[2 * wp() + dk + dj * nz()]; }
};

constexpr int round_up4(int x) { return (x + 3) / 4 * 4; }
constexpr int gcd_int(int a, int b) { return b == 0 ? a : gcd_int(b, a % b); }

// A two-element LDS block aligned to ALIGN elements.
template <typename CT, int ALIGN> using lds_pair = vec_at<CT, 2, ALIGN * (int)sizeof(CT)>;

// LDS reads for point O (0 or 1) of a pair of consecutive points: every read
// is a two-element block starting an even number of elements from the pair's
// first point, and the two points' identical loads are shared.  With a
// compile-time even height the pair's window index is even, so each block is
// one aligned read (8 or 16 bytes per lane, so lanes at an 8- or 16-byte
// stride hit the LDS banks without conflicts); ALIGN = 1 states that blocks
// are only aligned to an element.
template <typename CT, int WPAD, int ALIGN, int O>
struct PairAcc {
    const CT* const* row;   // rows j-1, j, j+1 of slot 0, field u at the pair's window index
    int sm, sc, sp;         // slots of planes i-1, i, i+1 (compile-time after inlining)
    template <int F, int dk, int dj, int di>
    __device__ __forceinline__ CT get() const {
        constexpr int e = O + dk;                              // -1 .. 2 from the pair start
        constexpr int start = e < 0 ? -2 : (e >= 2 ? 2 : 0);   // two-element block
        using V2 = typename lds_pair<CT, ALIGN>::type;
        const int slot = di < 0 ? sm : (di > 0 ? sp : sc);
        const V2 val = *reinterpret_cast<const V2*>(row[dj + 1] + (3 * slot + F) * WPAD + start);
        return val[e - start];
    }
    template <int dk, int dj, int di> __device__ __forceinline__ CT u() const { return get<0, dk, dj, di>(); }
    template <int dk, int dj, int di> __device__ __forceinline__ CT v() const { return get<1, dk, dj, di>(); }
    template <int dk, int dj, int di> __device__ __forceinline__ CT w() const { return get<2, dk, dj, di>(); }
};

// Planes held in the LDS ring: four for FP32 compute (one barrier per plane),
// three for FP64, whose larger slots would otherwise cost occupancy.
template <typename CT> constexpr int march_slots() { return sizeof(CT) == 4 ? 4 : 3; }

// The two-element blocks a pair of points reads: field F, row offset dj,
// plane offset di, block b in {-2, 0, 2} elements from the pair's start.  The
// stencil's reads (pw_point) per (field, dj, di) as a mask of level offsets
// dk (bit 0: dk = -1, bit 1: dk = 0, bit 2: dk = +1); a read at dk touches
// block -2 (dk = -1, first point), block 0 (every dk) and block 2 (dk = +1,
// second point).
constexpr int pair_dk_mask(int F, int dj, int di) {
    // [field][dj + 1][di + 1]
    constexpr int mask[3][3][3] = {{{0, 2, 0}, {6, 7, 2}, {2, 2, 0}},    // u
                                   {{0, 6, 2}, {2, 7, 2}, {0, 2, 0}},    // v
                                   {{0, 2, 0}, {2, 7, 3}, {0, 3, 0}}};   // w
    return mask[F][dj + 1][di + 1];
}
constexpr bool pair_block_used(int F, int dj, int di, int b) {
    return b == -2 ? (pair_dk_mask(F, dj, di) & 1) != 0
                   : (b == 0 ? pair_dk_mask(F, dj, di) != 0 : (pair_dk_mask(F, dj, di) & 4) != 0);
}
constexpr int pair_key(int F, int dj, int di, int b) { return ((F * 3 + dj + 1) * 3 + di + 1) * 3 + b / 2 + 1; }
constexpr int pair_carry_key(int F, int dj, int b) { return (F * 3 + dj + 1) * 3 + b / 2 + 1; }

// Pair reads from blocks already held in registers (indexed by pair_key).
template <typename CT, typename V2, int O>
struct CachedPairAcc {
    const V2* blk;
    template <int F, int dk, int dj, int di>
    __device__ __forceinline__ CT get() const {
        constexpr int e = O + dk;
        constexpr int start = e < 0 ? -2 : (e >= 2 ? 2 : 0);
        static_assert(pair_block_used(F, dj, di, start), "block missing from the pair block table");
        return blk[pair_key(F, dj, di, start)][e - start];
    }
    template <int dk, int dj, int di> __device__ __forceinline__ CT u() const { return get<0, dk, dj, di>(); }
    template <int dk, int dj, int di> __device__ __forceinline__ CT v() const { return get<1, dk, dj, di>(); }
    template <int dk, int dj, int di> __device__ __forceinline__ CT w() const { return get<2, dk, dj, di>(); }
};

// ---------------------------------------------------------------------------
// direct variant
// ---------------------------------------------------------------------------

// One lane takes a pair of levels (2m + 1, 2m + 2) of a column and walks along
// x through a segment of planes.  Nothing is staged in LDS: the pair's levels
// in the rows j-1, j, j+1 of u, v, w are loaded once per plane (nine loads of
// two levels) and kept in registers while the march needs them, at di = +1, 0
// and -1; the level below the pair and the one above it come from the
// neighbouring lanes (DPP wave shifts), so a wave computes 62 pairs and its
// first and last lane only load.  The loads of the next step are issued before
// the arithmetic of this one.  Bound by the vector memory instructions per
// point and by the loads in flight (one plane per wave).
//
// OFF: type of a byte offset within a plane.  uint32_t (planes below 2 GiB):
// buffer loads and stores off a scalar plane base, and lanes without a point
// store at the end of the buffer (the plane), which the hardware drops, so no
// branch hides the number of outstanding loads from the compiler.
// ODD: columns of odd height; their last pair has one level (its loads start
// one level early), and every level is stored by itself.
template <typename ST, typename OFF, bool ODD>
struct DirectPair {
    using CT = typename compute_of<ST>::type;
    using AR = typename arith_of<ST>::type;
    using V2 = typename lds_pair<CT, 2>::type;
    static constexpr bool NARROW = std::is_same<OFF, uint32_t>::value;
    static constexpr int E = (int)sizeof(ST);
    struct Raw {
        ST e[2];
    };
    const DomainArgs& d;
    OFF off[3];      // byte offset in a plane of the pair's loads in rows j-1, j, j+1
    OFF out[2];      // byte offset of the stores (ODD: of each level; NARROW: beyond the plane if there is none)
    bool live[2];    // the lane computes this level
    bool one;        // ODD: the last pair, one level
    int k0;          // the pair's first level
    uint32_t bytes;  // NARROW: bytes of a plane
    CT hx[3], hy[3], zc[2][6];
    Raw raw[27];     // pairs of the next step by pair_carry_key(F, dj, 0)
    V2 cm[27], c0[27];
    CT xs[2][2];

    // Plane offset at which a step first reads the pair of field F, row dj.
    static constexpr int ahead(int F, int dj) { return pair_block_used(F, dj, 1, 0) ? 1 : 0; }

    __device__ __forceinline__ DirectPair(const DomainArgs& dd, int64_t g, bool inner) : d(dd) {
        const int pairs = (d.nz + 1) / 2;
        const int64_t total = (int64_t)d.ny * pairs;
        const bool in = inner && g >= 0 && g < total;
        g = g < 0 ? 0 : (g < total ? g : total - 1);
        const int j = (int)(g / pairs) + 1;
        k0 = 2 * (int)(g % pairs) + 1;
        one = ODD && k0 == d.nz;
        const int lev = one ? k0 - 2 : k0 - 1;   // 0-based first level loaded
#pragma unroll
        for (int r = 0; r < 3; ++r) off[r] = (OFF)(((int64_t)(j + r - 1) * d.sy + lev) * E);
        bytes = NARROW ? (uint32_t)(((int64_t)d.ny + 2) * d.sy * E) : 0u;
        live[0] = in;
        live[1] = in && !one;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            out[q] = (OFF)(((int64_t)j * d.sy + k0 - 1 + q) * E);
            if (NARROW && !live[q]) out[q] = (OFF)bytes;
        }
#pragma unroll
        for (int f = 0; f < 3; ++f) {
            hx[f] = static_cast<CT>(d.cx[f]);
            hy[f] = static_cast<CT>(d.cy[f]);
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const PointCoefs<CT> c = point_coefs<ST>(d, min(k0 + q, d.nz));
            zc[q][0] = c.z1u;
            zc[q][1] = c.z2u;
            zc[q][2] = c.z1v;
            zc[q][3] = c.z2v;
            zc[q][4] = c.z1w;
            zc[q][5] = c.z2w;
        }
    }

    __device__ __forceinline__ int64_t plane_bytes(int i) const { return (int64_t)i * d.sx * E; }
    __device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(void* f, int i) const {
        constexpr int kRaw = 0x00027000;   // untyped, stride 0, no swizzle
        return __builtin_amdgcn_make_buffer_rsrc(static_cast<char*>(f) + plane_bytes(i), 0, (int)bytes, kRaw);
    }
    template <int F, int dj>
    __device__ __forceinline__ Raw load(int i) const {
        Raw r;
        const void* f = F == 0 ? d.u : (F == 1 ? d.v : d.w);
        if constexpr (NARROW) {
            const __amdgpu_buffer_rsrc_t b = buffer(const_cast<void*>(f), i);
            if constexpr (E == 8) {
                const auto x = __builtin_amdgcn_raw_buffer_load_b128(b, off[dj + 1], 0, 0);
                __builtin_memcpy(&r, &x, 16);
            } else if constexpr (E == 4) {
                const auto x = __builtin_amdgcn_raw_buffer_load_b64(b, off[dj + 1], 0, 0);
                __builtin_memcpy(&r, &x, 8);
            } else {
                const auto x = __builtin_amdgcn_raw_buffer_load_b32(b, off[dj + 1], 0, 0);
                __builtin_memcpy(&r, &x, 4);
            }
        } else {
            using V = typename vec_at<uint32_t, E == 2 ? 1 : 2 * E / 4, E>::type;
            const V x = *reinterpret_cast<global_ptr<const V>>(as_global(static_cast<const char*>(f) + plane_bytes(i)) + off[dj + 1]);
            __builtin_memcpy(&r, &x, sizeof(Raw));
        }
        return r;
    }
    // The pair in the compute type; the one level of a last odd pair comes first.
    __device__ __forceinline__ V2 widen(const Raw& r) const {
        const V2 v = V2{to_compute(r.e[0]), to_compute(r.e[1])};
        return ODD && one ? V2{v[1], v[1]} : v;
    }

    // Value of the lane below (wave_shr:1) or above (wave_shl:1); the first
    // and last lane, which have none, keep their own and do not store.
    template <int CTRL>
    static __device__ __forceinline__ float shift(float x) {
        return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(x), __float_as_int(x), CTRL, 0xf, 0xf, false));
    }
    template <int CTRL>
    static __device__ __forceinline__ double shift(double x) {
        const uint64_t u = (uint64_t)__double_as_longlong(x);
        const int lo = (int)(uint32_t)u, hi = (int)(uint32_t)(u >> 32);
        const uint32_t a = (uint32_t)__builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false);
        const uint32_t b = (uint32_t)__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false);
        return __longlong_as_double((long long)(((uint64_t)b << 32) | a));
    }
    // Block b of the pair whose own levels are v (only the level next to the
    // pair is read of an outer block).
    template <int b>
    static __device__ __forceinline__ V2 outer(const V2& v) {
        constexpr int kShr = 0x138, kShl = 0x130;
        const CT x = b < 0 ? shift<kShr>(v[1]) : shift<kShl>(v[0]);
        return V2{x, x};
    }

    // Issue the loads of step i.
    template <int K>
    __device__ __forceinline__ void load_step(int i) {
        if constexpr (K < 9) {
            constexpr int F = K / 3, dj = K % 3 - 1;
            raw[pair_carry_key(F, dj, 0)] = load<F, dj>(i + ahead(F, dj));
            load_step<K + 1>(i);
        }
    }
    // This step's blocks, from the loads, the carried registers and the neighbouring lanes.
    template <int K>
    __device__ __forceinline__ void gather(V2* blk) const {
        if constexpr (K < 54) {   // first the pairs themselves (b = 0), then the outer blocks
            constexpr bool own = K < 27;
            constexpr int F = (K % 27) / 9, dj = (K / 3) % 3 - 1, di = K % 3 - 1;
            if constexpr (own && pair_block_used(F, dj, di, 0)) {
                constexpr int key = pair_key(F, dj, di, 0);
                static_assert(di != -1 || pair_block_used(F, dj, 0, 0), "a pair of plane i-1 that was not read at plane i-1");
                if constexpr (di == ahead(F, dj)) blk[key] = widen(raw[pair_carry_key(F, dj, 0)]);
                else blk[key] = di == -1 ? cm[pair_carry_key(F, dj, 0)] : c0[pair_carry_key(F, dj, 0)];
            }
            if constexpr (!own) {
                if constexpr (pair_block_used(F, dj, di, -2)) gather_outer<F, dj, di, -2>(blk);
                if constexpr (pair_block_used(F, dj, di, 2)) gather_outer<F, dj, di, 2>(blk);
            }
            gather<K + 1>(blk);
        }
    }
    template <int F, int dj, int di, int b>
    __device__ __forceinline__ void gather_outer(V2* blk) const {
        constexpr int key = pair_key(F, dj, di, b);
        if constexpr (di == -1) blk[key] = cm[pair_carry_key(F, dj, b)];
        else if constexpr (di == 0 && pair_block_used(F, dj, 1, b)) blk[key] = c0[pair_carry_key(F, dj, b)];
        else blk[key] = outer<b>(blk[pair_key(F, dj, di, 0)]);
    }
    // Keep this step's blocks that the next step reads again.
    template <int K>
    __device__ __forceinline__ void keep(const V2* blk) {
        if constexpr (K < 27) {
            constexpr int F = K / 9, dj = (K / 3) % 3 - 1, b = (K % 3 - 1) * 2;
            if constexpr (pair_block_used(F, dj, -1, b)) cm[K] = blk[pair_key(F, dj, 0, b)];
            if constexpr (pair_block_used(F, dj, 0, b) && pair_block_used(F, dj, 1, b)) c0[K] = blk[pair_key(F, dj, 1, b)];
            keep<K + 1>(blk);
        }
    }
    // Carried blocks before step i: planes i-1 and i.
    template <int K>
    __device__ __forceinline__ void prime(int i) {
        if constexpr (K < 9) {
            constexpr int F = K / 3, dj = K % 3 - 1;
            constexpr int k0_ = pair_carry_key(F, dj, 0), km = pair_carry_key(F, dj, -2), kp = pair_carry_key(F, dj, 2);
            if constexpr (pair_block_used(F, dj, -1, 0)) cm[k0_] = widen(load<F, dj>(i - 1));
            if constexpr (ahead(F, dj) == 1) c0[k0_] = widen(load<F, dj>(i));
            if constexpr (pair_block_used(F, dj, -1, -2)) cm[km] = outer<-2>(cm[k0_]);
            if constexpr (pair_block_used(F, dj, -1, 2)) cm[kp] = outer<2>(cm[k0_]);
            if constexpr (pair_block_used(F, dj, 0, -2) && pair_block_used(F, dj, 1, -2)) c0[km] = outer<-2>(c0[k0_]);
            if constexpr (pair_block_used(F, dj, 0, 2) && pair_block_used(F, dj, 1, 2)) c0[kp] = outer<2>(c0[k0_]);
            prime<K + 1>(i);
        }
    }

    __device__ __forceinline__ void store(void* f, int i, CT a, CT b) const {
        if constexpr (NARROW) {
            constexpr int kNt = 2;   // non-temporal, as the march kernel's stores
            const __amdgpu_buffer_rsrc_t r = buffer(f, i);
            const Raw x{{from_compute<ST>(a), from_compute<ST>(b)}};
            if constexpr (ODD) {
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    if constexpr (E == 8) {
                        typename vec_at<uint32_t, 2, 8>::type w;
                        __builtin_memcpy(&w, &x.e[q], 8);
                        __builtin_amdgcn_raw_buffer_store_b64(w, r, out[q], 0, kNt);
                    } else if constexpr (E == 4) {
                        uint32_t w;
                        __builtin_memcpy(&w, &x.e[q], 4);
                        __builtin_amdgcn_raw_buffer_store_b32(w, r, out[q], 0, kNt);
                    } else {
                        uint16_t w;
                        __builtin_memcpy(&w, &x.e[q], 2);
                        __builtin_amdgcn_raw_buffer_store_b16(w, r, out[q], 0, kNt);
                    }
                }
            } else if constexpr (E == 8) {
                typename vec_at<uint32_t, 4, 16>::type w;
                __builtin_memcpy(&w, &x, 16);
                __builtin_amdgcn_raw_buffer_store_b128(w, r, out[0], 0, kNt);
            } else if constexpr (E == 4) {
                typename vec_at<uint32_t, 2, 8>::type w;
                __builtin_memcpy(&w, &x, 8);
                __builtin_amdgcn_raw_buffer_store_b64(w, r, out[0], 0, kNt);
            } else {
                uint32_t w;
                __builtin_memcpy(&w, &x, 4);
                __builtin_amdgcn_raw_buffer_store_b32(w, r, out[0], 0, kNt);
            }
        } else {
            const auto p = as_global(static_cast<char*>(f) + plane_bytes(i));
            if (live[0]) store_out<ST>(reinterpret_cast<global_ptr<ST>>(p + out[0]), a);
            if (live[1]) store_out<ST>(reinterpret_cast<global_ptr<ST>>(p + out[1]), b);
        }
    }

    __device__ __forceinline__ void run(int i_begin, int i_end) {
        load_step<0>(i_begin);
        prime<0>(i_begin);
        const V2 a = cm[pair_carry_key(0, 0, 0)], up = cm[pair_carry_key(0, 0, 2)], r = cm[pair_carry_key(0, 1, 0)];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            xs[q][0] = a[q] + r[q];                      // u(k, j) + u(k, j+1) of plane i_begin - 1
            xs[q][1] = a[q] + (q == 0 ? a[1] : up[0]);   // u(k) + u(k+1)
        }
        for (int i = i_begin; i <= i_end; ++i) {
            V2 blk[81];
            gather<0>(blk);
            load_step<0>(min(i + 1, i_end));   // the last step loads again what it has: no branch, exact waits
            CT res[2][3];
            const PointCoefs<CT> c0q{hx[0], hy[0], zc[0][0], zc[0][1], hy[1], hx[1],
                                     zc[0][2], zc[0][3], hx[2], hy[2], zc[0][4], zc[0][5]};
            const PointCoefs<CT> c1q{hx[0], hy[0], zc[1][0], zc[1][1], hy[1], hx[1],
                                     zc[1][2], zc[1][3], hx[2], hy[2], zc[1][4], zc[1][5]};
            CachedPairAcc<CT, V2, 0> A{blk};
            pw_point<AR, true, true, ODD>(A, k0, d.nz, c0q, res[0][0], res[0][1], res[0][2], xs[0]);
            CachedPairAcc<CT, V2, 1> B{blk};
            pw_point<AR, true, false, true>(B, k0 + 1, d.nz, c1q, res[1][0], res[1][1], res[1][2], xs[1]);
            keep<0>(blk);
            store(d.su, i, res[0][0], res[1][0]);
            store(d.sv, i, res[0][1], res[1][1]);
            store(d.sw, i, res[0][2], res[1][2]);
        }
    }
};

// One (chunk, segment) tile of the march: chunk c of the interior (j, k) run,
// planes i_begin .. i_end.  Every thread of the workgroup must run it (it
// holds barriers); `lds` must hold 3 * march_slots<CT>() * march_wpad(P, NZ)
// compute-type elements.
//
// NZ > 0: the domain's nz equals NZ, and every plane and the vectors in it are
// aligned to 16 bytes.
//
// NZ < 0: any height up to -NZ (a height class), any element alignment.  A
// window is a run of elements whatever the height, so it is still moved in
// whole vectors, at element alignment (the hardware takes 8- and 16-byte
// accesses at any dword for the same number of cache lines, 16-bit pairs at
// any halfword); the last vector of a window that is no multiple of VW starts
// early and overlaps the one before it.  EVEN (an even height): pairs of
// points are pairs of levels, aligned in LDS.  Otherwise a pair may straddle
// two columns, so both points select their bottom and top results, LDS reads
// are only aligned to an element, and a last chunk of an odd number of points
// ends with a pair that starts one point early (same values stored twice).
constexpr int march_wpad(int p, int nz) { return round_up4(p + 2 * (nz > 0 ? nz : -nz)); }
template <typename ST, int NT, int P, int NZ, bool EVEN = true, int DIST = 2, bool FORCE_EXACT = false>
struct MarchTile {
    using CT = typename compute_of<ST>::type;
    // Elements per load: as many as fill 16 bytes of LDS in the compute type,
    // so each lane's write of a converted vector is one conflict-free 16-byte
    // store (16-bit and int32 storage then load 8 bytes per lane).
    static constexpr int VW = int(16 / sizeof(CT));
    static constexpr int WPAD = march_wpad(P, NZ);                         // LDS elements per field and slot
    static constexpr int NVR = (3 * (WPAD / VW) + NT - 1) / NT;            // load rounds per thread (3 fields)
    static constexpr int PPT = P / NT;                                     // points per thread
    static constexpr bool RT = NZ < 0;                                     // run-time height, element alignment
    static constexpr bool PAIR = P % (2 * NT) == 0;
    static_assert(RT || (NZ % 2 == 0 && EVEN), "pairs of levels need an even compiled height");
    static constexpr bool ANY = RT && !EVEN;                               // pairs may straddle columns
    // Branch-free data movement (see the constructor) where storage is
    // narrower than the compute type: those kernels are bound by instruction
    // issue, and exact load counting lets two planes stay in flight.  FP32
    // and FP64 storage are bound by HBM and keep the branches, which cost
    // fewer registers (measured: 4% faster for them, 4-23% slower for the
    // converting types).
    static constexpr bool EXACT = FORCE_EXACT || sizeof(ST) < sizeof(CT);
    // Load rounds that every wave takes.  A window of 96 or 128 levels fills
    // two rounds and a sixteenth or a quarter of a third (four-element
    // vectors; FP64 compute four and an eighth or a half of a fifth): those
    // later rounds are left to the waves that hold part of the window, by a
    // branch uniform over the wave, if at most half of the waves do (NZ > 0)
    // or always (run-time heights).  1024 x 1000 x 96 int16 267 -> 262 us, the
    // 384-domain batch FP64 1097 -> 1086 us.
    static constexpr int LEAST = NZ > 0 ? NZ                                // least height of the kernel
                                 : (NZ == -kHeightClass[0] ? 2 : (NZ == -kHeightClass[1] ? kHeightClass[0] : kHeightClass[1]) + 1);
    static constexpr int VECS = 3 * ((P + 2 * LEAST + VW - 1) / VW);        // vectors of a full window at that height
    static constexpr int NFULL = !EXACT ? NVR : (NZ > 0 && (VECS % NT == 0 || VECS % NT > NT / 2) ? NVR : VECS / NT);
    // points past the chunk's end repeat its last ones (below)
    static constexpr bool CLAMP = EXACT || RT;
    static constexpr int NSLOT = march_slots<CT>();                       // planes in the LDS ring
    static_assert(VW * sizeof(ST) == 16 || VW * sizeof(ST) == 8, "8- or 16-byte loads");
    using Raw = typename std::conditional<VW * sizeof(ST) == 16, uint4, uint2>::type;
    static constexpr int RAW_ALIGN = RT ? int(sizeof(ST)) : int(sizeof(Raw));
    static constexpr int PAIR_ALIGN = ANY ? 1 : 2;   // elements a pair's window index is a multiple of
    // bytes an LDS write of a vector is aligned to
    static constexpr int PUT_ALIGN = !RT ? 16 : (ANY ? int(sizeof(CT)) : int(2 * sizeof(CT)));
    using V2 = typename lds_pair<CT, PAIR_ALIGN>::type;
    static_assert(P % NT == 0, "P must be a multiple of the block size");

    const DomainArgs& d;
    CT* lds;
    int nz_rt, wb, wlen;
    int li[PPT];
    int kk[PPT];
    bool live[PPT];          // point lies in the chunk (always true when CLAMP)
    CT hx[3], hy[3];       // uniform x and y coefficients of su, sv, sw
    CT zc[PPT][6];         // per-level vertical coefficients of each point
    // CARRY (with the branch-free data movement): blocks read at plane i as
    // "this plane" or "next plane" are kept in registers and reused at plane
    // i+1 as "previous plane" or "this plane", so a pair reads 17 of its 27
    // blocks from LDS instead of all of them.  cm: blocks for di = -1, c0:
    // blocks for di = 0, both indexed by pair_carry_key.  (FP32 storage,
    // bound by HBM, measured 4% slower with it: the carried registers cost a
    // resident workgroup per CU.)
    static constexpr bool CARRY = PAIR && EXACT;
    V2 cm[CARRY ? PPT / 2 : 1][27];
    V2 c0[CARRY ? PPT / 2 : 1][27];
    // CARRY: the x-face sums of sv's and sw's x terms, carried from plane to
    // plane (pw_point's xs), so each is formed once instead of twice
    CT xs[CARRY ? PPT : 1][2];
    // ZEND (fixed-point storage with the register carry, policies where a
    // zero product is an exact zero): the column's end points get zero
    // coefficients instead of selects -- all of them at k = 1, and at the top
    // the upper vertical coefficients of su and sv and the horizontal ones of
    // sw (tzd1, tzd2 are zero there already).  With finite operands that gives
    // a zero at k = 1, the column-top forms at k = nz and sw(nz) = 0; the zero
    // may carry either sign, which the integer output does not keep.  Floating
    // storage keeps the selects: its k = 1 outputs are +0 bit for bit, and no
    // value above the column top (level 1 of the next column) can reach a
    // result through 0 x Inf.  ph: per-point copies of the horizontal
    // coefficients xu, yu, yv, xv, xw, yw.
    static constexpr bool ZEND = CARRY && arith_of<ST>::type::kExactZeroFlux && is_fixed_point<ST>;
    CT ph[ZEND ? PPT : 1][6];
    // Rows j-1, j, j+1 at each pair's window index in slot 0, field u: with a
    // compile-time height one address and two immediates.
    const CT* row[PAIR ? PPT / 2 : 1][3];
    // The window vectors of all three fields are spread over the workgroup:
    // round r of this thread moves vector t + r NT -- field fsel[r] (-1: none),
    // element pointer gp[r] into the window of the next plane to load, LDS
    // offset loff[r].  Planes are loaded in order, so each load advances gp
    // by one plane (a 64-bit add of a uniform stride instead of a multiply).
    int fsel[NVR];
    global_ptr<const char> gp[NVR];
    int loff[NVR];
    bool more[NVR];   // rounds from NFULL on: this wave holds part of the window (uniform over the wave)
    // DIST planes in flight: plane p lives in register set (p - i_begin + 1) % DIST
    static_assert(DIST == 2 || DIST == 3, "two or three planes in flight");
    static constexpr int UNROLL = NSLOT * DIST / gcd_int(NSLOT, DIST);   // steps until slots and sets repeat
    static_assert(UNROLL <= 6, "unrolled block too long");
    Raw st[DIST][NVR];

    __device__ __forceinline__ int nz() const { return NZ > 0 ? NZ : nz_rt; }
    static constexpr int SLOT = 3 * WPAD;   // elements of one ring slot

    __device__ __forceinline__ MarchTile(const DomainArgs& dd, int c, CT* l) : d(dd), lds(l), nz_rt(dd.nz) {
        const int n = nz();
        const ChunkSpan cs = chunk_span(c, P, d.ny, n, ANY && PAIR);
        wb = cs.first - n;                              // window start: one column of y halo
        wlen = min(P + 2 * n, (d.ny + 2) * n - wb);
        const int nvec = (wlen + VW - 1) / VW;   // vectors per field (wlen >= 5 >= VW; NZ > 0: a multiple of VW)
#pragma unroll
        for (int r = 0; r < NVR; ++r) {
            // EXACT: the lanes past the window wrap round and move a
            // duplicate of an early vector (identical data to the same LDS
            // place), so loads and LDS writes need no branch and the compiler
            // can count outstanding loads exactly instead of waiting for all.
            const int v = EXACT ? ((int)threadIdx.x + r * NT) % (3 * nvec) : (int)threadIdx.x + r * NT;
            const int f = v < 3 * nvec ? v / nvec : -1;
            int q = (v - (f < 0 ? 0 : f) * nvec) * VW;
            if (RT) q = f < 0 ? 0 : min(q, wlen - VW);
            fsel[r] = f;
            more[r] = (int)__builtin_amdgcn_readfirstlane(threadIdx.x) + r * NT < 3 * nvec;
            const ST* base = static_cast<const ST*>(f == 0 ? d.u : (f == 1 ? d.v : d.w));
            gp[r] = as_global(reinterpret_cast<const char*>(base + (wb + q)));   // plane 0
            loff[r] = (f < 0 ? 0 : f) * WPAD + q;
        }
#pragma unroll
        for (int q = 0; q < PPT; ++q) {
            const int t = (int)threadIdx.x;
            int p = PAIR ? 2 * (t + NT * (q / 2)) + (q % 2) : t + NT * q;   // relative to cs.first
            // CLAMP: points past the chunk's end (last chunk of a domain)
            // recompute the chunk's last point or pair and store the
            // identical result again, so stores need no branch either.
            if (CLAMP) p = PAIR ? min(p, cs.count - 2 + (q % 2)) : min(p, cs.count - 1);
            live[q] = p < cs.count;
            kk[q] = point_level(cs.first, p, n);
            li[q] = p + n;
            const PointCoefs<CT> c = point_coefs<ST>(d, live[q] ? kk[q] : 1);
            zc[q][0] = c.z1u;
            zc[q][1] = c.z2u;
            zc[q][2] = c.z1v;
            zc[q][3] = c.z2v;
            zc[q][4] = c.z1w;
            zc[q][5] = c.z2w;
        }
        if constexpr (PAIR) {
#pragma unroll
            for (int pq = 0; pq < PPT / 2; ++pq)
#pragma unroll
                for (int dj = -1; dj <= 1; ++dj) row[pq][dj + 1] = lds + li[2 * pq] + dj * n;
        }
#pragma unroll
        for (int f = 0; f < 3; ++f) {
            hx[f] = static_cast<CT>(d.cx[f]);
            hy[f] = static_cast<CT>(d.cy[f]);
        }
        if constexpr (ZEND) {
#pragma unroll
            for (int q = 0; q < PPT; ++q) {
                const CT h[6] = {hx[0], hy[0], hy[1], hx[1], hx[2], hy[2]};
                // even heights: the first level of a pair is odd, the second even
                const bool bottom = (ANY || q % 2 == 0) && kk[q] == 1;
                const bool top = (ANY || q % 2 == 1) && kk[q] == nz();
#pragma unroll
                for (int e = 0; e < 6; ++e) ph[q][e] = (bottom || (top && e >= 4)) ? CT(0) : h[e];
                if (bottom) {
#pragma unroll
                    for (int e = 0; e < 6; ++e) zc[q][e] = CT(0);
                }
                if (top) {
                    zc[q][1] = CT(0);   // tzc2 of su
                    zc[q][3] = CT(0);   // tzc2 of sv
                }
            }
        }
    }

    // Move the load pointers to plane ip.
    __device__ __forceinline__ void seek(int64_t ip) {
        const int64_t po = ip * d.sx * (int64_t)sizeof(ST);
#pragma unroll
        for (int r = 0; r < NVR; ++r) gp[r] += po;
    }
    // Issue the global loads of the window of the next plane into `dst`.
    __device__ __forceinline__ void load_next(Raw* dst) {
        const int64_t ps = d.sx * (int64_t)sizeof(ST);   // uniform plane stride in bytes
        // the rounds of some waves first, so that the waits of the others
        // count the loads after theirs exactly
#pragma unroll
        for (int v = 0; v < NVR; ++v) {
            const int r = EXACT && NFULL < NVR ? NVR - 1 - v : v;
            if (EXACT ? r < NFULL || more[r] : fsel[r] >= 0) dst[r] = load_global<Raw, RAW_ALIGN>(gp[r]);
            gp[r] += ps;
        }
    }

    // Convert staged values to the compute type and write them to a slot.
    __device__ __forceinline__ void put_from(const Raw* src, int sidx) {
        CT* slot = lds + sidx * SLOT;
#pragma unroll
        for (int r = 0; r < NVR; ++r) {
            if (EXACT ? r < NFULL || more[r] : fsel[r] >= 0) {
                union {
                    Raw raw;
                    ST e[VW];
                } cv;
                cv.raw = src[r];
                CT out[VW];
                if constexpr (std::is_same<ST, bf16_t>::value) {
                    // a BF16 value is the upper half of its FP32 value: per
                    // 32-bit word, shift the low element up, mask the high one
                    uint32_t wd[sizeof(Raw) / 4];
                    __builtin_memcpy(wd, &cv.raw, sizeof(Raw));
#pragma unroll
                    for (int n = 0; n < VW / 2; ++n) {
                        out[2 * n] = __uint_as_float(wd[n] << 16);
                        out[2 * n + 1] = __uint_as_float(wd[n] & 0xffff0000u);
                    }
                } else {
#pragma unroll
                    for (int n = 0; n < VW; ++n) out[n] = to_compute(cv.e[n]);
                }
                static_assert(VW * sizeof(CT) == 16, "one 16-byte LDS write per vector");
                using V4 = typename vec_at<uint32_t, 4, PUT_ALIGN>::type;
                V4 x;
                __builtin_memcpy(&x, out, 16);
                *reinterpret_cast<V4*>(slot + loff[r]) = x;
            }
        }
    }

    // Block b of field F, row dj, of ring slot `slot` around pair pq.
    __device__ __forceinline__ V2 lds_block(int pq, int slot, int F, int dj, int b) const {
        return *reinterpret_cast<const V2*>(row[pq][dj + 1] + slot * SLOT + F * WPAD + b);
    }

    // CARRY: this step's blocks of pair pq, from the carried registers where
    // the previous step read them, else from LDS (slots sm, sc, sp hold planes
    // i-1, i, i+1).  Compile-time loop over all 81 keys; unused keys vanish.
    // Each LDS read is a single read (8 bytes for FP32 compute, 16 for FP64) at
    // an immediate offset from the pair's base address -- one with a compiled
    // height, one per row otherwise; every slot and field lies within the
    // 64 KiB offset range.  A scheduling barrier after each read keeps the
    // compiler from pairing reads into two-address reads, whose 2 KiB offset
    // range would cost a vector add for a new base address nearly every
    // time: in these VALU-bound kernels five such adds per plane and thread
    // measured slower than the extra LDS instructions.
    template <int K>
    __device__ __forceinline__ void gather_blocks(V2* blk, int pq, int sm, int sc, int sp) {
        if constexpr (K < 81) {
            constexpr int F = K / 27, dj = (K / 9) % 3 - 1, di = (K / 3) % 3 - 1, b = (K % 3 - 1) * 2;
            if constexpr (pair_block_used(F, dj, di, b)) {
                if constexpr (di == -1 && pair_block_used(F, dj, 0, b)) {
                    blk[K] = cm[pq][pair_carry_key(F, dj, b)];
                } else if constexpr (di == 0 && pair_block_used(F, dj, 1, b)) {
                    blk[K] = c0[pq][pair_carry_key(F, dj, b)];
                } else {
                    const int slot = di < 0 ? sm : (di > 0 ? sp : sc);
                    blk[K] = lds_block(pq, slot, F, dj, b);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            gather_blocks<K + 1>(blk, pq, sm, sc, sp);
        }
    }
    // CARRY: keep this step's blocks that the next step reuses.
    template <int K>
    __device__ __forceinline__ void keep_blocks(const V2* blk, int pq) {
        if constexpr (K < 27) {
            constexpr int F = K / 9, dj = (K / 3) % 3 - 1, b = (K % 3 - 1) * 2;
            if constexpr (pair_block_used(F, dj, -1, b) && pair_block_used(F, dj, 0, b))
                cm[pq][K] = blk[pair_key(F, dj, 0, b)];
            if constexpr (pair_block_used(F, dj, 0, b) && pair_block_used(F, dj, 1, b))
                c0[pq][K] = blk[pair_key(F, dj, 1, b)];
            keep_blocks<K + 1>(blk, pq);
        }
    }
    // CARRY: before a tile's first step, load the carried blocks from planes
    // i_begin - 1 (slot 0) and i_begin (slot 1).
    template <int K>
    __device__ __forceinline__ void prime_blocks(int pq) {
        if constexpr (K < 27) {
            constexpr int F = K / 9, dj = (K / 3) % 3 - 1, b = (K % 3 - 1) * 2;
            if constexpr (pair_block_used(F, dj, -1, b) && pair_block_used(F, dj, 0, b))
                cm[pq][K] = lds_block(pq, 0, F, dj, b);
            if constexpr (pair_block_used(F, dj, 0, b) && pair_block_used(F, dj, 1, b))
                c0[pq][K] = lds_block(pq, 1, F, dj, b);
            prime_blocks<K + 1>(pq);
        }
    }

    // CARRY: the x-face sums at plane i_begin - 1 from the carried blocks of
    // that plane (cm, just primed), in the order pw_point forms them.
    __device__ __forceinline__ void prime_sums(int pq) {
        constexpr int kU0 = pair_carry_key(0, 0, 0), kU0b = pair_carry_key(0, 0, 2), kU1 = pair_carry_key(0, 1, 0);
        static_assert(pair_block_used(0, 0, -1, 0) && pair_block_used(0, 0, 0, 0) && pair_block_used(0, 0, -1, 2) &&
                          pair_block_used(0, 0, 0, 2) && pair_block_used(0, 1, -1, 0) && pair_block_used(0, 1, 0, 0),
                      "sum blocks must be carried");
        const V2 a = cm[pq][kU0], b = cm[pq][kU0b], r = cm[pq][kU1];
        xs[2 * pq][0] = a[0] + r[0];       // u(k, j) + u(k, j+1)
        xs[2 * pq][1] = a[0] + a[1];       // u(k) + u(k+1)
        xs[2 * pq + 1][0] = a[1] + r[1];
        xs[2 * pq + 1][1] = a[1] + b[0];
    }

    // Compute plane i from the slots sm (plane i-1), sc (plane i), sp (plane i+1).
    __device__ __forceinline__ void compute(int i, int sm, int sc, int sp) {
        const int64_t obase = (int64_t)i * d.sx + wb;
        using AR = typename arith_of<ST>::type;
        CT res[PPT][3];
        V2 blk[CARRY ? PPT / 2 : 1][81];   // CARRY: this step's blocks, indexed by pair_key
#pragma unroll
        for (int q = 0; q < PPT; ++q) {
            const int l = li[q];
            const PointCoefs<CT> c = ZEND ? PointCoefs<CT>{ph[q][0], ph[q][1], zc[q][0], zc[q][1],
                                                           ph[q][2], ph[q][3], zc[q][2], zc[q][3],
                                                           ph[q][4], ph[q][5], zc[q][4], zc[q][5]}
                                          : PointCoefs<CT>{hx[0], hy[0], zc[q][0], zc[q][1], hy[1], hx[1],
                                                           zc[q][2], zc[q][3], hx[2], hy[2], zc[q][4], zc[q][5]};
            if constexpr (CARRY) {
                if (q % 2 == 0) gather_blocks<0>(blk[q / 2], q / 2, sm, sc, sp);
                if (q % 2 == 0) {
                    CachedPairAcc<CT, V2, 0> A{blk[q / 2]};
                    pw_point<AR, false, !ZEND, ANY && !ZEND>(A, kk[q], nz(), c, res[q][0], res[q][1], res[q][2], xs[q]);
                } else {
                    CachedPairAcc<CT, V2, 1> A{blk[q / 2]};
                    pw_point<AR, false, ANY && !ZEND, !ZEND>(A, kk[q], nz(), c, res[q][0], res[q][1], res[q][2], xs[q]);
                    keep_blocks<0>(blk[q / 2], q / 2);
                }
            } else if constexpr (PAIR) {
                // even heights: the pair's first level is odd (k = 1 possible,
                // never the top); the second is even (never k = 1, the top
                // possible)
                if (q % 2 == 0) {
                    PairAcc<CT, WPAD, PAIR_ALIGN, 0> A{row[q / 2], sm, sc, sp};
                    pw_point<AR, false, true, ANY>(A, kk[q], nz(), c, res[q][0], res[q][1], res[q][2]);
                } else {
                    PairAcc<CT, WPAD, PAIR_ALIGN, 1> A{row[q / 2], sm, sc, sp};
                    pw_point<AR, false, ANY, true>(A, kk[q], nz(), c, res[q][0], res[q][1], res[q][2]);
                }
            } else {
                LdsAcc<CT, NZ, WPAD> A{lds + sm * SLOT + l, lds + sc * SLOT + l, lds + sp * SLOT + l, nz_rt};
                pw_point<AR, false>(A, kk[q], nz(), c, res[q][0], res[q][1], res[q][2]);
            }
        }
        global_ptr<ST> outs[3] = {as_global(static_cast<ST*>(d.su) + obase), as_global(static_cast<ST*>(d.sv) + obase),
                                  as_global(static_cast<ST*>(d.sw) + obase)};
        if constexpr (PAIR) {
#pragma unroll
            for (int q = 0; q < PPT; q += 2) {
                if (!CLAMP && !live[q]) continue;   // NZ > 0: a pair never straddles the chunk end (P, nz even)
#pragma unroll
                for (int f = 0; f < 3; ++f) store_pair<ST, RT ? 1 : 2>(outs[f] + (uint32_t)li[q], res[q][f], res[q + 1][f]);
            }
        } else {
#pragma unroll
            for (int q = 0; q < PPT; ++q) {
                if (!CLAMP && !live[q]) continue;
#pragma unroll
                for (int f = 0; f < 3; ++f) store_out(outs[f] + (uint32_t)li[q], res[q][f]);
            }
        }
    }

    // One march step: publish plane i+1, prefetch plane i+1+DIST, compute
    // plane i.  DIST register sets keep DIST planes in flight, so each load
    // has DIST steps to arrive; SET = (i - i_begin) % DIST holds plane i+1
    // and then receives plane i+1+DIST.  With three slots the slot of plane
    // i-1 is refilled by the next step, so a second barrier keeps it until
    // every wave has computed plane i; with four slots that refill happens
    // one step later, behind the next step's barrier, and one barrier per
    // plane suffices.
    template <int SET>
    __device__ __forceinline__ void step(int i, int i_end, int sm, int sc, int sp) {
        put_from(st[SET], sp);
        __syncthreads();
        if (i + 1 + DIST <= i_end + 1) load_next(st[SET]);   // plane i + 1 + DIST
        compute(i, sm, sc, sp);
        if constexpr (NSLOT == 3) __syncthreads();
    }

    // Steps R .. UNROLL-1 of one unrolled block starting at plane i; slots and
    // register sets are compile-time constants.  Returns false past i_end.
    template <int R>
    __device__ __forceinline__ bool block(int i, int i_end) {
        if constexpr (R == UNROLL) {
            return true;
        } else {
            if (i + R > i_end) return false;
            step<R % DIST>(i + R, i_end, R % NSLOT, (R + 1) % NSLOT, (R + 2) % NSLOT);
            return block<R + 1>(i, i_end);
        }
    }

    __device__ __forceinline__ void run(int i_begin, int i_end) {
        // the first planes are requested together, so a tile's start waits
        // for one memory latency, not several
        {
            // planes i_begin - 1, i_begin, i_begin + 1 (<= nx + 1, always
            // there), then up to i_begin + DIST; the steps continue in order
            // with plane i + 1 + DIST, and once one plane lies past i_end + 1
            // every later one does too
            Raw a[NVR], b[NVR];
            seek((int64_t)(i_begin - 1));
            load_next(a);
            load_next(b);
            load_next(st[0]);
#pragma unroll
            for (int q = 1; q < DIST; ++q) {
                if (i_begin + 1 + q <= i_end + 1) load_next(st[q]);
            }
            put_from(a, 0);
            put_from(b, 1);
        }
        if constexpr (CARRY) {
            __syncthreads();
#pragma unroll
            for (int pq = 0; pq < PPT / 2; ++pq) {
                prime_blocks<0>(pq);
                prime_sums(pq);
            }
        }
        for (int i = i_begin;; i += UNROLL) {
            if (!block<0>(i, i_end)) break;
        }
        // the next tile of a persistent workgroup refills slots 0 and 1
        if constexpr (NSLOT == 4) __syncthreads();
    }
};

template <typename ST, int NT, int P, int NZ, bool EVEN = true, int DIST = 2, bool FORCE_EXACT = false>
__device__ __forceinline__ void march_tile(const DomainArgs& d, int c, int i_begin, int i_end,
                                           typename compute_of<ST>::type* lds) {
    MarchTile<ST, NT, P, NZ, EVEN, DIST, FORCE_EXACT> t(d, c, lds);
    t.run(i_begin, i_end);
}

// Resident waves per SIMD the single-domain march kernel may reach: FP64
// storage is held at two (two workgroups per CU, each with two planes in
// flight): three workgroups per CU, with more planes in flight or without,
// measured 10% slower on 2048 x 2048 x 64 -- more concurrent streams cost
// the HBM more than the extra bytes in flight gain.  Other storage types are
// not capped.
template <typename ST> constexpr int march_max_waves() { return std::is_same<ST, double>::value ? 2 : 8; }

// Single domain: the (chunk, segment) tile of this workgroup, false if none.
__device__ __forceinline__ bool single_tile(const MarchGeom& g, int nx, int& c, int& i_begin, int& i_end) {
    const int tile = g.run > 0 ? march_compact_tile((int)blockIdx.x, g.nchunks * g.nseg, g.run, g.blocks)
                               : xcd_tile((int)blockIdx.x, (int)gridDim.x);
    if (tile < 0) return false;   // whole workgroup
    const int s = tile / g.nchunks;
    c = tile - s * g.nchunks;
    i_begin = 1 + s * g.seg;
    i_end = min(i_begin + g.seg - 1, nx);
    return true;
}

// Direct variant: 62 pairs of levels per wave, any workgroup of whole waves.
constexpr int kDirectPairs = 62;
template <typename ST, typename OFF, bool ODD>
__global__ __launch_bounds__(512) void pw_direct_kernel(DomainArgs d, MarchGeom g) {
    int c, i_begin, i_end;
    if (!single_tile(g, d.nx, c, i_begin, i_end)) return;
    const int waves = (int)blockDim.x / 64, wave = (int)threadIdx.x / 64, lane = (int)threadIdx.x % 64;
    const int64_t first = ((int64_t)c * waves + wave) * kDirectPairs;
    DirectPair<ST, OFF, ODD> p(d, first + lane - 1, lane >= 1 && lane <= kDirectPairs);
    p.run(i_begin, i_end);
}

// March variant: one workgroup per (chunk, segment) tile.
template <typename ST, int NT, int P, int NZ, bool EVEN>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(1, march_max_waves<ST>())))
void pw_march_kernel(DomainArgs d, MarchGeom g) {
    using CT = typename compute_of<ST>::type;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    CT* lds = reinterpret_cast<CT*>(smem_raw);
    int c, i_begin, i_end;
    if (!single_tile(g, d.nx, c, i_begin, i_end)) return;
    march_tile<ST, NT, P, NZ, EVEN>(d, c, i_begin, i_end, lds);
}

}  // namespace pw
