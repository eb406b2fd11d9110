// Device-side building blocks of the point rasterizer for gfx950 (MI355X),
// shared by the one-view kernels (rz_kernels.hip), the multi-view batch
// kernels (rz_batch.hip), the general point-size and float-depth kernels
// (rz_general.hip), the screen-sorted path (rz_sorted.hip) and the
// reciprocal self-check (rz_check.hip).
//
// Method: Schuetz & Wimmer, "Rendering Point Clouds with Compute Shaders"
// (arXiv 1908.02681), section 2.1 (atomicMin rasterization, resolve/clear)
// and section 2.2 (high-quality splatting).
//
// Every file that includes this header must be compiled with
// -ffp-contract=off; the pragma below repeats it, so that the projection is
// the exact IEEE operation sequence stated in include/rz.h (fused
// multiply-adds only where written as such, correctly rounded f32 division,
// no flush of denormals).
//
// Code style rule for the point kernels: decisions are kept in separate
// boolean flags computed with selects; no element of a register array is
// updated inside a divergent branch.  This hipcc build was seen to
// mis-allocate that form (the reject copy of a phi was hoisted above the
// branch and overwritten).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rz.h"
#include "rz_internal.h"

#pragma clang fp contract(off)

namespace rz {
namespace dev {

constexpr double kQMax = 1099511627774.0;   // 2^40 - 2
constexpr int kXcds = 8;                     // XCDs of an MI355X
constexpr int kMaxWaves = 512 / 64;
constexpr uint32_t kMaxPixel = 32767;        // of a row or column: screens have at most 2^15
constexpr uint32_t kTileMin = 4096;          // workgroup tile of the depth pass: 32 KiB
constexpr uint32_t kTileHq = 2048;           // workgroup tile of the accumulate pass: 32 KiB
constexpr uint32_t kWaveTileWords = 1024;    // per-wave tile: 8 KiB of LDS
constexpr uint32_t kWaveTileMin = kWaveTileWords;   // pixels (one key each)
// The small per-wave tile (2 KiB): a quarter of the LDS per wave, so that
// LDS no longer caps the waves per SIMD of kernels with few registers
// (measured: the multi-view kernels at 4 points per thread).
constexpr uint32_t kWaveTileSmallWords = 256;

// Tiling modes of the point kernels.  kBinWaveSmall is kBinWave with the
// small tile: the kernels take the tile size as an argument, so both modes
// share the kBinWave code.
// kBinGroup (not a launch option) is kBinWaveSmall in a workgroup of kGroupWaves waves,
// which share their tiles where they cover the same pixels.
enum : int { kBinNone = 0, kBinBlock = 1, kBinWave = 2, kBinWaveSmall = 3, kBinGroup = 4 };
constexpr uint32_t kGroupWaves = 4;
static_assert(kSmallTune.block == 64 * kGroupWaves && kUnreadTune.block == kSmallTune.block,
              "small clouds' workgroups");

// Words of one wave's tile in a per-wave tiling mode.  The accumulate pass's
// small tile has 6 KiB: three words a pixel (two copies of the sums and the
// window's threshold) for the 256 pixels of the depth pass's.
__host__ __device__ constexpr uint32_t wave_tile_words(int bin, bool hq)
{
    return bin != kBinWaveSmall ? kWaveTileWords
           : hq                 ? 3 * kWaveTileSmallWords
                                : kWaveTileSmallWords;
}

// Four points of a plane.  The hardware's 16-byte loads need no more than
// dword alignment, so planes cut anywhere out of larger ones take them too.
typedef float f32x4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));

// Device memory and LDS as such: pointers that come out of a table are
// otherwise taken through flat instructions, which occupy both paths.
typedef __attribute__((address_space(1))) uint64_t gu64;
typedef __attribute__((address_space(3))) uint64_t lu64;
typedef __attribute__((address_space(3))) u64x2 lu64x2;
__device__ __forceinline__ gu64 *global_ptr(const uint64_t *p) { return (gu64 *)p; }
// LDS by its byte address: LDS addresses are 32 bits, so that a tile's origin
// folds into its base.
__device__ __forceinline__ uint32_t lds_addr(const uint64_t *p)
{
    return (uint32_t)(uintptr_t)(lu64 *)p;
}
__device__ __forceinline__ lu64 *lds_ptr(uint32_t a) { return (lu64 *)(uintptr_t)a; }
__device__ __forceinline__ lu64x2 *lds_ptr2(uint32_t a) { return (lu64x2 *)(uintptr_t)a; }

// Streaming (non-temporal) access: the data is touched once per pass.
template <typename T>
__device__ __forceinline__ T ldnt(const T *p) { return __builtin_nontemporal_load(p); }
template <typename T>
__device__ __forceinline__ void stnt(T v, T *p) { __builtin_nontemporal_store(v, p); }

// 0 <= t < 2^52, integral: t + 2^52 is exact and its 52 mantissa bits are t.
__device__ __forceinline__ uint64_t to_u64(double t)
{
    return (uint64_t)__double_as_longlong(t + 0x1p52) & 0xFFFFFFFFFFFFFull;
}

// True when the predicate holds on any active lane of the wave: the ballot
// mask itself (HIP's __any goes through an int and costs two more vector
// instructions per call).
__device__ __forceinline__ bool wave_any(bool p) { return __builtin_amdgcn_ballot_w64(p) != 0; }

// Piecewise depth map (section 2.1, sub-ranges with their own precision):
// range k with start rb[k] <= d < rb[k+1]; q = rbase[k] + floor((d - rb[k]) *
// rs[k]), which stays below rbase[k+1] because IEEE rounding is monotone.
__device__ __forceinline__ uint64_t piecewise_q(const Proj &P, double d)
{
    int k = 0;
    for (int i = 1; i < 8; ++i)
        k = (i < P.nr && d >= P.rb[i]) ? i : k;
    const double tf = floor((d - P.rb[k]) * P.rs[k]);
    const uint64_t q = P.rbase[k] + to_u64(tf);
    return q > (1ull << 40) - 2 ? (1ull << 40) - 2 : q;
}

// Linear depth of integer depth q under the piecewise map.
__device__ __forceinline__ double piecewise_depth(const Proj &P, uint64_t q)
{
    int k = 0;
    for (int i = 1; i < 8; ++i)
        k = (i < P.nr && q >= P.rbase[i]) ? i : k;
    return P.rb[k] + (double)(q - P.rbase[k]) * P.rinv[k];
}

// Section 2.2's window: does a fragment of depth q join the pixel whose
// nearest depth is qmin?  Linear maps: exact integer test; piecewise maps:
// the linear depths the integers stand for, in double precision.
template <bool PW>
__device__ __forceinline__ bool in_window(const Proj &P, uint32_t eps_num, uint32_t eps_den,
                                          uint64_t q, uint64_t qmin)
{
    if (!PW || P.nr == 0)   // PW kernels also serve linear views of a batch
        return (uint64_t)eps_den * (q - qmin) <= (uint64_t)eps_num * (qmin + P.z0);
    const double dq = piecewise_depth(P, q);
    const double dm = piecewise_depth(P, qmin);
    const double lhs = (double)eps_den * (dq - dm);
    const double rhs = (double)eps_num * dm;
    return lhs <= rhs;
}

// Integer depth below 2^52 as a double (exact): its bits under the
// exponent of 2^52, minus 2^52.
__device__ __forceinline__ double int52_to_double(uint64_t v)
{
    return __longlong_as_double((long long)(v | 0x4330000000000000ull)) - 0x1p52;
}

// live && in_window, for the accumulate passes.  Linear maps with z0 < 2^52
// decide in double precision first: D = q - qmin and S = qmin + z0 are
// exact there, den * D and num * S are each rounded once, and rounding is
// monotone, so when the rounded products differ they order the exact ones
// the same way.  Only equal rounded products (a fragment on the window's
// edge) take the integer test, in a branch a wave enters only when one of
// its live lanes needs it.  Same result as in_window for every input; the
// 64-bit integer products it avoids are quarter-rate instructions.
template <bool PW>
__device__ __forceinline__ bool in_window_live(const Proj &P, uint32_t eps_num, uint32_t eps_den,
                                               uint64_t q, uint64_t qmin, bool live)
{
    if ((PW && P.nr != 0) || !P.wfp)
        return live && in_window<PW>(P, eps_num, eps_den, q, qmin);
    const double dm = int52_to_double(qmin);
    const double lhs = (double)eps_den * (int52_to_double(q) - dm);
    const double rhs = (double)eps_num * (dm + P.z0d);
    bool ok = live & (lhs < rhs);
    const bool edge = live & (lhs == rhs);
    if (wave_any(edge)) {
        const bool ex = (uint64_t)eps_den * (q - qmin) <= (uint64_t)eps_num * (qmin + P.z0);
        ok = edge ? ex : ok;
    }
    return ok;
}

// The window as a threshold per pixel, for the linear and scale maps:
// den * (q - qmin) <= num * S with S = qmin + z0 holds exactly for the integers
// q <= qmin + floor(num * S / den).  num * S stays below 2^50 for the eps and z0
// of window_exact, so that the product, the remainder of the estimated quotient
// and with it the corrected floor are exact.
__device__ __forceinline__ bool window_exact(const Proj &P, const Eps &eps)
{
    return eps.num <= 256u && eps.den <= 4096u && P.z0 <= (1ull << 41);
}

__device__ __forceinline__ double window_threshold(const Proj &P, const Eps &eps, uint64_t key)
{
    const double den = (double)eps.den;
    const double dm = int52_to_double(key >> 24);
    const double r = (double)eps.num * (dm + P.z0d);
    const double f = floor(r * eps.inv_den);
    const double rem = __builtin_fma(-f, den, r);
    const double off = rem < 0.0 ? -1.0 : rem >= den ? 1.0 : 0.0;
    return dm + (f + off);
}

// The IEEE quotient 1 / w for w > 0, without the full division sequence:
// one Newton-Raphson correction of the hardware estimate, r + r * (1 - w r)
// with both steps fused (Markstein's method).  Run over every positive
// float on gfx950, it equals the correctly rounded reciprocal for all w in
// [2^-126, 2^126) and misses only for denormal w, w >= 2^126 and +inf;
// those lanes take the division.  For w <= 0 or NaN the value is never
// used (every caller culls the point), so it is left as it comes.
__device__ __forceinline__ float recip_newton(float w)
{
    const float r = __builtin_amdgcn_rcpf(w);
    const float e = __builtin_fmaf(-w, r, 1.0f);
    return __builtin_fmaf(r, e, r);
}

__device__ __forceinline__ float recip_rn(float w)
{
    float f = recip_newton(w);
    const bool slow = (w > 0.0f) & ((w < 0x1p-126f) | (w >= 0x1p126f));
    if (wave_any(slow)) {   // wave-uniform; no lane needs it in practice
        const float q = 1.0f / w;
        f = slow ? q : f;
    }
    return f;
}

// Translation column of the float matrix (clip x, y, w) and of the depth
// row in double, the addend of the first fused step of each row.
// lane_trans() returns it as per-lane values (moves that the compiler cannot
// fold back), made once per chunk: a fused multiply-add can take only one scalar-register operand
// on gfx950, so with the scalar copies every row of every point would need
// a move first.
struct Trans {
    float tx, ty, tw;
    double td;   // the depth row's translation (double precision)
};

__device__ __forceinline__ float lane_copy(float v)
{
    float r;
    asm("v_mov_b32_e32 %0, %1" : "=v"(r) : "s"(v));
    return r;
}

__device__ __forceinline__ double lane_copy(double v)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = __float_as_uint(lane_copy(__uint_as_float((uint32_t)b)));
    const uint32_t hi = __float_as_uint(lane_copy(__uint_as_float((uint32_t)(b >> 32))));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

__device__ __forceinline__ Trans lane_trans(const Proj &P)
{
    return Trans{lane_copy(P.m[3]), lane_copy(P.m[7]), lane_copy(P.m[11]), lane_copy(P.v[3])};
}

__device__ __forceinline__ Trans scalar_trans(const Proj &P)
{
    return Trans{P.m[3], P.m[7], P.m[11], P.v[3]};
}

// Pixel of one point (section 2.1's projection in single precision: each
// clip coordinate a chain of fused multiply-adds from the translation
// column through the x, y and z terms), its clip w and 1 / w (rounded once;
// x and y are scaled by it, as a perspective divide does, and the viewport
// maps them with one fused scale and offset).  Returns false when the point
// is culled (w <= 0 or off screen).
// Straight-line code: the pixel of a culled point is 0, never a conversion
// of an out-of-range float.
__device__ __forceinline__ bool project(const Proj &P, const Trans &T, float x, float y, float z,
                                        uint32_t &px, uint32_t &py, float &cw, float &iw)
{
    float cx = __builtin_fmaf(P.m[0], x, T.tx);
    cx = __builtin_fmaf(P.m[1], y, cx);
    cx = __builtin_fmaf(P.m[2], z, cx);
    float cy = __builtin_fmaf(P.m[4], x, T.ty);
    cy = __builtin_fmaf(P.m[5], y, cy);
    cy = __builtin_fmaf(P.m[6], z, cy);
    cw = __builtin_fmaf(P.m[8], x, T.tw);
    cw = __builtin_fmaf(P.m[9], y, cw);
    cw = __builtin_fmaf(P.m[10], z, cw);
    iw = recip_rn(cw);
    const float nx = cx * iw;
    const float ny = cy * iw;
    const float fx = __builtin_fmaf(nx, P.hw, P.hw);   // viewport: scale and offset
    const float fy = __builtin_fmaf(ny, P.hh, P.hh);
    const bool vis = (cw > 0.0f) & (fx >= 0.0f) & (fx < P.fw) & (fy >= 0.0f) & (fy < P.fh);
    px = (uint32_t)(int32_t)(vis ? fx : 0.0f);
    py = (uint32_t)(int32_t)(vis ? fy : 0.0f);
    return vis;
}

// Depth in double precision (section 1, section 2.1): row 3 of VP, fused
// in the same order as the clip coordinates.
__device__ __forceinline__ double depth_of(const Proj &P, double td, float x, float y, float z)
{
    double d = __builtin_fma(P.v[0], (double)x, td);
    d = __builtin_fma(P.v[1], (double)y, d);
    d = __builtin_fma(P.v[2], (double)z, d);
    return d;
}

__device__ __forceinline__ double depth_of(const Proj &P, const Trans &T, float x, float y,
                                           float z)
{
    return depth_of(P, T.td, x, y, z);
}

// Depth of one point in any of the encodings, without the assumptions of a chunk
// (ChunkKey): clears `in` for a point outside [near, far) or clipped by the 24-bit
// window depth of the perspective matrix (RZ_DEPTH_GL24), whose depth is then
// meaningless.  ZK = 0 for the integer maps; cw and iw = 1 / cw are read by the
// float encodings only (RZ_DEPTH_F32REV: the complemented reversed float depth).
// Straight-line, and the 24-bit code is converted only from a value inside the window.
template <bool PW, int ZK>
__device__ __forceinline__ uint64_t depth_enc(const Proj &P, const Trans &T, float x, float y,
                                              float z, float cw, float iw, bool &in)
{
    const double d = depth_of(P, T, x, y, z);
    const bool in_range = (d >= P.near_) & (d < P.far_);
    in = in & in_range;
    if constexpr (ZK == 0) {
        if (PW && P.nr != 0)
            return piecewise_q(P, in_range ? d : P.near_);
        return to_u64(fmin(floor((d - P.o) * P.s), kQMax));   // d < near gives garbage, unused
    }
    if constexpr (ZK == RZ_DEPTH_F32REV)
        return 0xFFFFFFFFull - (uint64_t)__float_as_uint(P.nearf / cw);
    float cz = __builtin_fmaf(P.mz[0], x, P.mz[3]);
    cz = __builtin_fmaf(P.mz[1], y, cz);
    cz = __builtin_fmaf(P.mz[2], z, cz);
    const float nz = cz * iw;
    const bool clip = (nz >= -1.0f) & (nz <= 1.0f);
    in = in & clip;
    const float zw = (nz + 1.0f) * 0.5f;
    const float t = zw * 16777215.0f;
    return (uint64_t)(uint32_t)floor((double)(clip ? t : 0.0f) + 0.5);
}

// The fragment of one point: pixel coordinates and 40-bit depth (section
// 2.1) under an integer depth map (P.zkind == 0).  Returns false when the point is
// discarded; q is then meaningless.  PW = false: linear or scale map
// only (P.nr == 0), so the piecewise tables are never read; PW = true serves
// every integer map.  Straight-line code apart from one wave-uniform skip
// of the depth when no lane of the wave is on screen.
// vis: the point is on screen (w > 0, inside the framebuffer), whatever its
// depth.
template <bool PW>
__device__ __forceinline__ bool fragment(const Proj &P, const Trans &T, float x, float y, float z,
                                         uint32_t &px, uint32_t &py, uint64_t &q, bool &vis)
{
    float cw, iw;
    vis = project(P, T, x, y, z, px, py, cw, iw);
    q = 0;
    bool in = vis;
    if (!wave_any(vis))
        return false;
    q = depth_enc<PW, 0>(P, T, x, y, z, cw, iw, in);
    return in;
}

template <bool PW>
__device__ __forceinline__ bool fragment(const Proj &P, const Trans &T, float x, float y, float z,
                                         uint32_t &px, uint32_t &py, uint64_t &q)
{
    bool vis;
    return fragment<PW>(P, T, x, y, z, px, py, q, vis);
}

template <bool PW>
__device__ __forceinline__ bool fragment(const Proj &P, float x, float y, float z,
                                         uint32_t &px, uint32_t &py, uint64_t &q)
{
    return fragment<PW>(P, scalar_trans(P), x, y, z, px, py, q);
}

// The fragment of one point in a float encoding (ZK).
template <int ZK>
__device__ __forceinline__ bool fragment_zk(const Proj &P, const Trans &T, float x, float y,
                                            float z, uint32_t &px, uint32_t &py, uint64_t &q)
{
    static_assert(ZK == RZ_DEPTH_GL24 || ZK == RZ_DEPTH_F32REV, "float encodings only");
    float cw, iw;
    bool in = project(P, T, x, y, z, px, py, cw, iw);
    q = 0;
    if (!wave_any(in))
        return false;
    q = depth_enc<false, ZK>(P, T, x, y, z, cw, iw, in);
    return in;
}

// The fragment of the kernels templated on the depth encoding: ZK = 0 for
// the integer maps, else RZ_DEPTH_GL24 or RZ_DEPTH_F32REV.
template <bool PW, int ZK>
__device__ __forceinline__ bool fragment_enc(const Proj &P, const Trans &T, float x, float y,
                                             float z, uint32_t &px, uint32_t &py, uint64_t &q)
{
    if constexpr (ZK == 0)
        return fragment<PW>(P, T, x, y, z, px, py, q);
    else
        return fragment_zk<ZK>(P, T, x, y, z, px, py, q);
}

// Workgroup -> chunk of points.  Workgroups are dealt round-robin to the 8
// XCDs; with the remap, XCD k works through the k-th eighth of the chunks,
// so spatially coherent (e.g. Morton-ordered) ranges share one L2.
template <bool XCD>
__device__ __forceinline__ int64_t chunk_index()
{
    const int64_t b = blockIdx.x;
    if (!XCD)
        return b;
    const int64_t per = gridDim.x / kXcds;   // grid is a multiple of 8
    return (b % kXcds) * per + b / kXcds;
}

// Loads the PPT points of this thread.  Vector form: PPT/4 groups of four
// consecutive points, group g at chunk + g*4*blockDim + 4*tid, so every
// load instruction of a wave reads one contiguous 1 KiB span per plane,
// whatever the planes' alignment (a frame of a 6.25M-point slice that starts
// three elements into its planes: 75.6 us with single-element loads, 58.2 us
// with these).  Scalar form (tail chunk): same point indices, bounds checked
// one by one.
template <int PPT>
__device__ __forceinline__ bool chunk_full(const Pts &p, int64_t base)
{
    return base + 4 * (int64_t)blockDim.x * (PPT / 4) <= p.n;
}

template <int PPT>
__device__ __forceinline__ void load_full(const Pts &p, int64_t base, float (&x)[PPT],
                                          float (&y)[PPT], float (&z)[PPT], uint32_t (&c)[PPT])
{
    const int64_t stride = 4 * (int64_t)blockDim.x;
    const int64_t first = base + 4 * (int64_t)threadIdx.x;
#pragma unroll
    for (int g = 0; g < PPT / 4; ++g) {
        const int64_t i = first + g * stride;
        const f32x4 vx =
            __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(p.x + i));
        const f32x4 vy =
            __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(p.y + i));
        const f32x4 vz =
            __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(p.z + i));
        const u32x4 vc =
            __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p.rgb + i));
        x[4 * g + 0] = vx.x; x[4 * g + 1] = vx.y; x[4 * g + 2] = vx.z; x[4 * g + 3] = vx.w;
        y[4 * g + 0] = vy.x; y[4 * g + 1] = vy.y; y[4 * g + 2] = vy.z; y[4 * g + 3] = vy.w;
        z[4 * g + 0] = vz.x; z[4 * g + 1] = vz.y; z[4 * g + 2] = vz.z; z[4 * g + 3] = vz.w;
        c[4 * g + 0] = vc.x; c[4 * g + 1] = vc.y; c[4 * g + 2] = vc.z; c[4 * g + 3] = vc.w;
    }
}

// The loads of any chunk, for kernels that carry no per-point bounds flags: points
// past the end read as NaN, which every projection culls (a NaN coordinate
// makes clip w NaN, and w > 0 fails), so the chunk code is the same for the
// last chunk as for all others.
template <int PPT>
__device__ __forceinline__ void load_points_nan(const Pts &p, int64_t base, float (&x)[PPT],
                                                float (&y)[PPT], float (&z)[PPT],
                                                uint32_t (&c)[PPT])
{
    if (chunk_full<PPT>(p, base)) {
        load_full<PPT>(p, base, x, y, z, c);
        return;
    }
    const int64_t stride = 4 * (int64_t)blockDim.x;
    const int64_t first = base + 4 * (int64_t)threadIdx.x;
    const float nan = __builtin_nanf("");
#pragma unroll
    for (int g = 0; g < PPT / 4; ++g) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t i = first + g * stride + k;
            const bool ok = i < p.n;
            x[4 * g + k] = ok ? p.x[i] : nan;
            y[4 * g + k] = ok ? p.y[i] : nan;
            z[4 * g + k] = ok ? p.z[i] : nan;
            c[4 * g + k] = ok ? p.rgb[i] : 0u;
        }
    }
}

// Minimum over the 64 lanes of a wave with DPP moves (all lanes active):
// quads, 8-lane halves, 16-lane rows, then row broadcasts into lane 63.
__device__ __forceinline__ uint32_t wave_min(uint32_t v)
{
    // Each step moves a neighbour's value in by DPP and keeps the smaller.
    // Lanes the step does not write get the identity ~0, so the move folds
    // into the minimum (one v_min_u32 with a DPP operand per step).
#define RZ_DPP_MIN(ctrl, rows)                                                             \
    {                                                                                      \
        const uint32_t t = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, ctrl, rows,   \
                                                                 0xF, false);              \
        v = v < t ? v : t;                                                                 \
    }
    RZ_DPP_MIN(0xB1, 0xF)    // quad_perm [1,0,3,2]
    RZ_DPP_MIN(0x4E, 0xF)    // quad_perm [2,3,0,1]
    RZ_DPP_MIN(0x141, 0xF)   // row_half_mirror
    RZ_DPP_MIN(0x140, 0xF)   // row_mirror
    RZ_DPP_MIN(0x142, 0xA)   // row_bcast:15 into rows 1 and 3
    RZ_DPP_MIN(0x143, 0xC)   // row_bcast:31 into rows 2 and 3
#undef RZ_DPP_MIN
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// The same for the maximum (identity 0).
__device__ __forceinline__ uint32_t wave_max(uint32_t v)
{
#define RZ_DPP_MAX(ctrl, rows)                                                             \
    {                                                                                      \
        const uint32_t t = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, rows,    \
                                                                 0xF, false);              \
        v = v > t ? v : t;                                                                 \
    }
    RZ_DPP_MAX(0xB1, 0xF)
    RZ_DPP_MAX(0x4E, 0xF)
    RZ_DPP_MAX(0x141, 0xF)
    RZ_DPP_MAX(0x140, 0xF)
    RZ_DPP_MAX(0x142, 0xA)
    RZ_DPP_MAX(0x143, 0xC)
#undef RZ_DPP_MAX
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Screen rectangle of the live fragments of the workgroup.  Every thread
// must call it (it synchronises the workgroup); every thread gets the same
// answer.  Empty when x0 > x1.
struct Box {
    uint32_t x0, y0, x1, y1;
};

template <int PPT>
__device__ __forceinline__ Box block_box(const uint32_t (&px)[PPT], const uint32_t (&py)[PPT],
                                         const bool (&live)[PPT], uint32_t (*s_box)[4])
{
    uint32_t m[4] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu};
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
        const uint32_t a = live[j] ? px[j] : 0xFFFFFFFFu;
        const uint32_t b = live[j] ? py[j] : 0xFFFFFFFFu;
        const uint32_t c = live[j] ? ~px[j] : 0xFFFFFFFFu;
        const uint32_t d = live[j] ? ~py[j] : 0xFFFFFFFFu;
        m[0] = a < m[0] ? a : m[0];
        m[1] = b < m[1] ? b : m[1];
        m[2] = c < m[2] ? c : m[2];
        m[3] = d < m[3] ? d : m[3];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
        m[k] = wave_min(m[k]);
    const uint32_t wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            s_box[wave][k] = m[k];
    }
    __syncthreads();
    const uint32_t nw = blockDim.x >> 6;
    for (uint32_t w = 0; w < nw; ++w) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            m[k] = s_box[w][k] < m[k] ? s_box[w][k] : m[k];
    }
    return Box{m[0], m[1], ~m[2], ~m[3]};
}

// Depth pass over one chunk already in registers (section 2.1): every
// surviving fragment takes part in a 64-bit minimum per pixel of fb.  None
// of the refinements changes the result, because min is order independent
// and the framebuffer only decreases:
//  - consecutive fragments of a thread in one pixel are merged in registers;
//  - BIN: when the workgroup's fragments fall in a small screen rectangle,
//    they are merged with LDS atomics in a tile first, and the tile is
//    flushed row by row (coalesced global atomics, one per touched pixel);
//  - EARLY: the framebuffer is read first and the atomic skipped when it is
//    already <= the key (a stale read can only be larger than the true
//    value, so the skip is always safe).
// With BIN every thread of the workgroup must call it; it returns with the
// workgroup past its last barrier but threads possibly still flushing, so a
// caller that reuses s_tile or s_box must synchronise first.
template <int PPT, bool EARLY, bool BIN, bool PW>
__device__ __forceinline__ void raster_chunk(const Proj &P, uint64_t *__restrict__ fb,
                                             const float (&x)[PPT], const float (&y)[PPT],
                                             const float (&z)[PPT], const uint32_t (&c)[PPT],
                                             const bool (&in)[PPT], uint64_t *s_tile,
                                             uint32_t (*s_box)[4])
{
    uint32_t px[PPT], py[PPT], pix[PPT];
    uint64_t key[PPT];
    bool live[PPT];
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
        uint64_t q = 0;
        uint32_t a = 0, b = 0;
        live[j] = fragment<PW>(P, x[j], y[j], z[j], a, b, q) & in[j];
        px[j] = a;
        py[j] = b;
        pix[j] = __umul24(b, (uint32_t)P.width) + a;   // both below 2^15
        key[j] = (q << 24) | ((uint64_t)c[j] & kRgbMask);
    }
#pragma unroll
    for (int j = 1; j < PPT; ++j) {
        const bool same = live[j] && live[j - 1] && pix[j] == pix[j - 1];
        const uint64_t lo = key[j] < key[j - 1] ? key[j] : key[j - 1];
        key[j] = same ? lo : key[j];
        live[j - 1] = live[j - 1] && !same;
    }

    bool direct[PPT];
    Box box{1, 1, 0, 0};
    uint32_t bw = 0, bh = 0;
    bool tiled = false;
    if (BIN) {
        box = block_box<PPT>(px, py, live, s_box);
        if (box.x0 <= box.x1) {
            bw = box.x1 - box.x0 + 1;
            bh = box.y1 - box.y0 + 1;
            tiled = (uint64_t)bw * bh <= kTileMin;
        }
    }
    if (tiled) {
        const uint32_t area = bw * bh;
        for (uint32_t i = threadIdx.x; i < area; i += blockDim.x)
            s_tile[i] = ~0ull;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < PPT; ++j) {
            const uint32_t tx = px[j] - box.x0, ty = py[j] - box.y0;
            const bool inside = live[j] && tx < bw && ty < bh;
            direct[j] = live[j] && !inside;
            if (inside)
                __hip_atomic_fetch_min(&s_tile[ty * bw + tx], key[j], __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < area; i += blockDim.x) {
            const uint64_t v = s_tile[i];
            if (v != ~0ull) {
                const uint32_t r = i / bw;
                const uint32_t col = i - r * bw;
                uint64_t *dst = fb + (__umul24(box.y0 + r, (uint32_t)P.width) + box.x0 + col);
                const uint64_t cur = __hip_atomic_load(dst, __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_AGENT);
                if (v < cur)
                    __hip_atomic_fetch_min(dst, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    } else {
#pragma unroll
        for (int j = 0; j < PPT; ++j)
            direct[j] = live[j];
    }

    // fragments not merged in a tile go straight to the framebuffer
    if (EARLY) {
        uint64_t cur[PPT];
#pragma unroll
        for (int j = 0; j < PPT; ++j)
            cur[j] = __hip_atomic_load(fb + (direct[j] ? pix[j] : 0u), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int j = 0; j < PPT; ++j)
            if (direct[j] && key[j] < cur[j])
                __hip_atomic_fetch_min(fb + pix[j], key[j], __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
    } else {
#pragma unroll
        for (int j = 0; j < PPT; ++j)
            if (direct[j])
                __hip_atomic_fetch_min(fb + pix[j], key[j], __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Orders the LDS accesses of one wave: LDS executes a wave's instructions in
// issue order, so only the compiler has to be kept from moving them.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Row and column of tile entry i in a tile bw wide: i / bw through a float
// reciprocal, corrected to the exact quotient (i < 2^24, bw <= 2^15).
__device__ __forceinline__ void tile_rc(uint32_t i, uint32_t bw, float inv_bw, uint32_t &r,
                                        uint32_t &col)
{
    uint32_t q = (uint32_t)((float)i * inv_bw);
    q = __umul24(q, bw) > i ? q - 1 : q;          // products below 2^25
    q = __umul24(q + 1, bw) <= i ? q + 1 : q;
    r = q;
    col = i - __umul24(q, bw);
}

// Screen rectangle of the live fragments of one wave (no workgroup barrier).
template <int PPT>
__device__ __forceinline__ Box wave_box(const uint32_t (&px)[PPT], const uint32_t (&py)[PPT],
                                        const bool (&live)[PPT])
{
    static_assert(PPT % 2 == 0, "points are taken in pairs");
    uint32_t lx = 0xFFFFFFFFu, ly = 0xFFFFFFFFu, hx = 0u, hy = 0u;
#pragma unroll
    for (int j = 0; j < PPT; j += 2) {   // pairs: three-operand min and max
        const uint32_t a0 = live[j] ? px[j] : 0xFFFFFFFFu,
                       a1 = live[j + 1] ? px[j + 1] : 0xFFFFFFFFu;
        const uint32_t b0 = live[j] ? py[j] : 0xFFFFFFFFu,
                       b1 = live[j + 1] ? py[j + 1] : 0xFFFFFFFFu;
        const uint32_t c0 = live[j] ? px[j] : 0u, c1 = live[j + 1] ? px[j + 1] : 0u;
        const uint32_t d0 = live[j] ? py[j] : 0u, d1 = live[j + 1] ? py[j + 1] : 0u;
        lx = min(lx, min(a0, a1));
        ly = min(ly, min(b0, b1));
        hx = max(hx, max(c0, c1));
        hy = max(hy, max(d0, d1));
    }
    // no live lane: lx = ~0 > hx = 0, an empty box
    return Box{wave_min(lx), wave_min(ly), wave_max(hx), wave_max(hy)};
}

// A register of its own for v: keeps the compiler from carrying values that it
// derived from v over to here in further registers.
__device__ __forceinline__ void own(float &v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void own(uint32_t &v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void own(int32_t &v) { asm volatile("" : "+v"(v)); }

// The loads of v end here, whether v is used or not: a register with a load
// pending would make whatever takes it next wait for every memory operation
// since (one counter covers them all, in order).
__device__ __forceinline__ void arrive(uint64_t &v) { asm volatile("" : "+v"(v)); }

// Window position of one point without the cull and the IEEE division: the
// steps of project() with the corrected estimate of 1 / w, which is the IEEE
// quotient for w in [2^-126, 2^126).  (The matrix unit's 4x4x1 instruction
// gives the same bits for a whole column of rows and issues three instructions
// for nine here, but takes longer: a batch of 64 views of 100M points 17.2 ms
// with it, 16.2 ms with these.)
__device__ __forceinline__ void window_pos(const Proj &P, const Trans &T, float x, float y, float z,
                                           float &cw, float &fx, float &fy)
{
    float cx = __builtin_fmaf(P.m[0], x, T.tx);
    cx = __builtin_fmaf(P.m[1], y, cx);
    cx = __builtin_fmaf(P.m[2], z, cx);
    float cy = __builtin_fmaf(P.m[4], x, T.ty);
    cy = __builtin_fmaf(P.m[5], y, cy);
    cy = __builtin_fmaf(P.m[6], z, cy);
    cw = __builtin_fmaf(P.m[8], x, T.tw);
    cw = __builtin_fmaf(P.m[9], y, cw);
    cw = __builtin_fmaf(P.m[10], z, cw);
    const float iw = recip_newton(cw);
    fx = __builtin_fmaf(cx * iw, P.hw, P.hw);
    fy = __builtin_fmaf(cy * iw, P.hh, P.hh);
}

// Minimum within each row of 16 lanes.
__device__ __forceinline__ int32_t row_min(int32_t v)
{
#define RZ_DPP_ROW(ctrl)                                                                   \
    {                                                                                      \
        const int32_t t = __builtin_amdgcn_update_dpp(0x7FFFFFFF, v, ctrl, 0xF, 0xF, false); \
        v = v < t ? v : t;                                                                 \
    }
    RZ_DPP_ROW(0xB1)    // quad_perm [1,0,3,2]
    RZ_DPP_ROW(0x4E)    // quad_perm [2,3,0,1]
    RZ_DPP_ROW(0x141)   // row_half_mirror
    RZ_DPP_ROW(0x140)   // row_mirror
#undef RZ_DPP_ROW
    return v;
}

// Minima of x and y and the complements of their maxima over a wave, in the rows of
// 16 lanes: x's minimum, x's maximum, y's minimum, y's maximum.  The four reductions
// share their steps: two half-wave swaps leave x (rows 0, 1) beside y (rows 2, 3), a
// row swap puts the minima into the even rows and the complemented maxima into the
// odd ones, and one 16-lane reduction finishes all four: 11 instructions where four
// 64-lane reductions take 24.
__device__ __forceinline__ int32_t wave_bounds(int32_t xlo, int32_t xhi, int32_t ylo, int32_t yhi)
{
    // rows 0 and 1: x, rows 2 and 3: y
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)xlo, (uint32_t)ylo, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)~xhi, (uint32_t)~yhi, false, false);
    const int32_t l2 = min((int32_t)lo[0], (int32_t)lo[1]);
    const int32_t h2 = min((int32_t)hi[0], (int32_t)hi[1]);
    // rows 0 and 2: the minima, rows 1 and 3: the complements of the maxima
    const auto lh = __builtin_amdgcn_permlane16_swap((uint32_t)l2, (uint32_t)h2, false, false);
    return row_min(min((int32_t)lh[0], (int32_t)lh[1]));
}

// The rectangle of which wave_bounds() left the sides `v` in its rows.
__device__ __forceinline__ Box bounds_box(int32_t v)
{
    Box box;
    box.x0 = (uint32_t)__builtin_amdgcn_readlane(v, 0);
    box.x1 = (uint32_t)__builtin_amdgcn_readlane(v, 16);
    box.y0 = (uint32_t)__builtin_amdgcn_readlane(v, 32);
    box.y1 = (uint32_t)__builtin_amdgcn_readlane(v, 48);
    return box;
}

// Minimum and sum within each quad of lanes.
__device__ __forceinline__ uint32_t quad_min(uint32_t v)
{
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0xB1, 0xF, 0xF, false));
    return min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x4E, 0xF, 0xF, false));
}
__device__ __forceinline__ uint32_t quad_sum(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false);
    return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false);
}

// Window positions of a wave's points: kOnScreen, with their pixel rectangle,
// when every point of the wave has a w in [2^-126, 2^126) and an on-screen window
// position; kOffScreen when all lie beyond one edge of the screen or behind the
// camera (w negative or -0, which is never drawn); kEdge, with the on-screen part
// of their rectangle, when only w is known to be fine; kMixed (and the rest
// meaningless) otherwise.  The first two are nearly all chunks of an ordered cloud,
// and need no flag per point.  The tests run on bit patterns, where the order of
// non-negative floats is that of the integers and every other value (negative,
// NaN, infinite) falls outside: w through an unsigned minimum and maximum, x
// and y through signed ones.
enum Where { kOnScreen, kOffScreen, kEdge, kMixed };

template <int PPT>
__device__ __forceinline__ Where window_all(const Proj &P, const Trans &T, const float (&x)[PPT],
                                           const float (&y)[PPT], const float (&z)[PPT],
                                           float (&fx)[PPT], float (&fy)[PPT], Box &box)
{
    static_assert(PPT % 2 == 0, "points are taken in pairs");
    uint32_t wlo = ~0u, whi = 0u;
    int32_t xlo = 0x7FFFFFFF, ylo = 0x7FFFFFFF, xhi = -0x7FFFFFFF - 1, yhi = -0x7FFFFFFF - 1;
#pragma unroll
    for (int j = 0; j < PPT; j += 2) {   // pairs: three-operand min and max
        float w0, w1;
        window_pos(P, T, x[j], y[j], z[j], w0, fx[j], fy[j]);
        window_pos(P, T, x[j + 1], y[j + 1], z[j + 1], w1, fx[j + 1], fy[j + 1]);
        const uint32_t a = __float_as_uint(w0), b = __float_as_uint(w1);
        wlo = min(wlo, min(a, b));
        whi = max(whi, max(a, b));
        const int32_t x0 = __float_as_int(fx[j]), x1 = __float_as_int(fx[j + 1]);
        const int32_t y0 = __float_as_int(fy[j]), y1 = __float_as_int(fy[j + 1]);
        xlo = min(xlo, min(x0, x1));
        xhi = max(xhi, max(x0, x1));
        ylo = min(ylo, min(y0, y1));
        yhi = max(yhi, max(y0, y1));
        if (j % 4)
            __builtin_amdgcn_sched_barrier(0);
    }
    const int32_t m = wave_bounds(xlo, xhi, ylo, yhi);
    const uint32_t lane = threadIdx.x & 63u;
    const bool odd = (lane & 16u) != 0;
    const int32_t size = (lane & 32u) ? __float_as_int(P.fh) : __float_as_int(P.fw);
    if (wave_any((wlo < 0x00800000u) | (whi >= 0x7E800000u)))   // some w <= 0: all of them?
        return wave_any(wlo < 0x80000000u) ? kMixed : kOffScreen;
    // even rows: minimum >= 0; odd rows: maximum < size, on the complement
    const bool inside = m >= (odd ? -size : 0);
    if (wave_any(m >= (odd ? 0 : size)))   // a minimum >= size or a maximum < 0
        return kOffScreen;
    // the minima and maxima as pixels, cut at the screen's edge
    const float edge = odd ? __int_as_float(size) - 1.0f : 0.0f;
    const int32_t px = (int32_t)(inside ? __int_as_float(odd ? ~m : m) : edge);
    box = bounds_box(px);
    if (wave_any(!inside))
        return kEdge;
    return kOnScreen;
}

// A window position on screen.
__device__ __forceinline__ bool on_screen(const Proj &P, float fx, float fy)
{
    return (fx >= 0.0f) & (fx < P.fw) & (fy >= 0.0f) & (fy < P.fh);
}

// Clip w of one point, with no register shared with the projection's.
__device__ __forceinline__ float clip_w(const Proj &P, const Trans &T, float x, float y, float z)
{
    own(x), own(y), own(z);
    float cw = __builtin_fmaf(P.m[8], x, T.tw);
    cw = __builtin_fmaf(P.m[9], y, cw);
    return __builtin_fmaf(P.m[10], z, cw);
}

// After kMixed: bit j of `behind` set where the lane's point j has w <= 0 or NaN, so
// that its window position means nothing.  True when some point of the wave has a
// positive w outside [2^-126, 2^126): its position is not the one by the IEEE quotient.
template <int PPT>
__device__ __forceinline__ bool sort_w(const Proj &P, const Trans &T, const float (&x)[PPT],
                                       const float (&y)[PPT], const float (&z)[PPT],
                                       uint32_t &behind)
{
    bool slow = false;
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
        const float cw = clip_w(P, T, x[j], y[j], z[j]);
        slow = slow | ((cw > 0.0f) & ((cw < 0x1p-126f) | (cw >= 0x1p126f)));
        behind |= cw > 0.0f ? 0u : 1u << j;
        __builtin_amdgcn_sched_barrier(0);
    }
    return wave_any(slow);
}

// Whether a lane's point j is on screen, by its window position and `behind`.
__device__ __forceinline__ bool visible(const Proj &P, float fx, float fy, uint32_t behind, int j)
{
    return on_screen(P, fx, fy) & ((behind & (1u << j)) == 0u);
}

// Box of the on-screen points of a wave; without one, x1 lies beyond kMaxPixel.
template <int PPT>
__device__ __forceinline__ Box window_box(const Proj &P, const float (&fx)[PPT],
                                          const float (&fy)[PPT], uint32_t behind)
{
    int32_t xlo = 0x7FFFFFFF, ylo = 0x7FFFFFFF, xhi = -1, yhi = -1;
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
        float wx = fx[j], wy = fy[j];
        own(wx), own(wy);
        const bool vis = visible(P, wx, wy, behind, j);
        const int32_t px = (int32_t)(vis ? wx : 0.0f), py = (int32_t)(vis ? wy : 0.0f);
        xlo = min(xlo, vis ? px : 0x7FFFFFFF);
        ylo = min(ylo, vis ? py : 0x7FFFFFFF);
        xhi = max(xhi, vis ? px : -1);
        yhi = max(yhi, vis ? py : -1);
        // this point's work ends here, and with it its registers
        own(xlo), own(ylo), own(xhi), own(yhi);
    }
    const int32_t m = wave_bounds(xlo, xhi, ylo, yhi);
    return bounds_box((threadIdx.x & 16u) != 0 ? ~m : m);
}

// One uniform range of the depth map for a whole chunk: the linear and scale
// maps have one; of a piecewise map, the one that holds depth d of lane 0.
struct Range1 {
    double lo, hi;   // depths it serves without a clamp
    double o, s;     // q = base + floor((d - o) * s)
    uint64_t base;
};

template <bool PW>
__device__ __forceinline__ Range1 uniform_range(const Proj &P, double d)
{
    if (!PW || P.nr == 0)
        return Range1{P.dlo[0], P.dhi[0], P.o, P.s, 0ull};
    int k = 0;
    for (int i = 1; i < P.nr; ++i)
        k = d >= P.rb[i] ? i : k;
    k = __builtin_amdgcn_readfirstlane(k);
    return Range1{P.dlo[k], P.dhi[k], P.rb[k], P.rs[k], P.rbase[k]};
}

// q << 24 | rgb from floor((d - o) * s) + 2^52, whose mantissa is q: the key's
// high word is the shifted pair, its low word takes three bytes of colour.
__device__ __forceinline__ uint64_t make_key(uint64_t q52, uint32_t c)
{
    const uint32_t lo = (uint32_t)q52, hi = (uint32_t)(q52 >> 32);
    const uint32_t kh = __builtin_amdgcn_alignbyte(hi, lo, 1);
    const uint32_t kl = __builtin_amdgcn_perm(lo, c, 0x04020100u);
    return ((uint64_t)kh << 32) | kl;
}

// Keys of the points of one chunk, all of them with a w in [2^-126, 2^126).
// `in` is cleared by a point for which the key is not valid: one outside
// [near, far), outside the chunk's range of the depth map, or clipped by the
// 24-bit window depth.
template <bool PW, int ZK>
struct ChunkKey {
    const Proj &P;
    const Trans &T;
    Range1 R;

    // x, y, z: a point of the chunk, whose range serves for all
    __device__ __forceinline__ ChunkKey(const Proj &p, const Trans &t, float x, float y, float z)
        : P(p), T(t), R(uniform_range<PW>(p, PW ? depth_of(p, t.td, x, y, z) : 0.0))
    {
    }

    __device__ __forceinline__ uint64_t operator()(float x, float y, float z, uint32_t c,
                                                   bool &in) const
    {
        const double d = depth_of(P, T.td, x, y, z);
        in = in & (d >= R.lo) & (d < R.hi);
        if constexpr (ZK == 0) {
            const double f = floor((d - R.o) * R.s);
            uint64_t q52 = (uint64_t)__double_as_longlong(f + 0x1p52);
            if (PW)
                q52 += R.base;
            return make_key(q52, c);
        }
        float cw = __builtin_fmaf(P.m[8], x, T.tw);
        cw = __builtin_fmaf(P.m[9], y, cw);
        cw = __builtin_fmaf(P.m[10], z, cw);
        if constexpr (ZK == RZ_DEPTH_F32REV)
            return make_key(0xFFFFFFFFull - (uint64_t)__float_as_uint(P.nearf / cw), c);
        float cz = __builtin_fmaf(P.mz[0], x, P.mz[3]);
        cz = __builtin_fmaf(P.mz[1], y, cz);
        cz = __builtin_fmaf(P.mz[2], z, cz);
        const float nz = cz * recip_newton(cw);
        const bool clip = (nz >= -1.0f) & (nz <= 1.0f);
        in = in & clip;
        const float zw = (nz + 1.0f) * 0.5f;
        const float t = zw * 16777215.0f;
        return make_key((uint64_t)(uint32_t)floor((double)(clip ? t : 0.0f) + 0.5), c);
    }
};

// The screen rectangle of a wave's fragments as a tile in LDS.
struct WaveTile {
    uint32_t x0, y0, bw, area;
    float inv_bw;
    uint32_t width;
};

__device__ __forceinline__ WaveTile wave_tile(const Proj &P, const Box &box)
{
    WaveTile t;
    t.x0 = box.x0;
    t.y0 = box.y0;
    t.bw = box.x1 - box.x0 + 1;
    t.area = t.bw * (box.y1 - box.y0 + 1);   // both at most 2^15
    t.inv_bw = __builtin_amdgcn_rcpf((float)t.bw);   // tile_rc corrects it
    t.width = (uint32_t)P.width;
    return t;
}

// Pixel of entry i of the tile, in the framebuffer.
__device__ __forceinline__ uint32_t tile_pixel(const WaveTile &t, uint32_t i)
{
    uint32_t r, col;
    tile_rc(i, t.bw, t.inv_bw, r, col);
    return __umul24(t.y0 + r, t.width) + t.x0 + col;
}

// LDS address of a point's entry in a tile of 1 << sh bytes per pixel whose
// entry 0 lies at `first` - origin << sh (modulo 2^32).
__device__ __forceinline__ uint32_t tile_entry(const WaveTile &t, float fx, float fy, uint32_t sh,
                                               uint32_t first)
{
    return ((__umul24((uint32_t)(int32_t)fy, t.bw) + (uint32_t)(int32_t)fx) << sh) + first;
}

// `first` of a wave's tile at LDS address base: kept in one register.
__device__ __forceinline__ uint32_t tile_first(const WaveTile &t, uint32_t base, uint32_t sh)
{
    uint32_t v = base - ((t.y0 * t.bw + t.x0) << sh);
    asm("" : "+v"(v));
    return v;
}

// The nearest key of a pixel, for an early out.  With `l2` the read may be served
// by the XCD's L2, where a neighbouring chunk left the line; the key may be older
// then, but like any early one it is an upper bound (at its start a launch sees
// at least what the launches before it wrote).
__device__ __forceinline__ uint64_t read_nearest(const gu64 *p, bool l2)
{
    return l2 ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)
              : __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// What raster_chunk_wave leaves to be flushed: its tile (area 0: nothing), and
// of the lane's first entry the pixel and the nearest key read before.
struct MinFlush {
    WaveTile t;
    uint32_t p0;
    uint64_t cur;
    bool four;
};

// Nearest key of entry i of a tile at LDS address base, kept once or four times.
__device__ __forceinline__ uint64_t tile_nearest(uint32_t base, uint32_t i, bool four)
{
    if (!four)
        return *lds_ptr(base + 8 * i);
    const u64x2 a = *lds_ptr2(base + 32 * i), b = *lds_ptr2(base + 32 * i + 16);
    const uint64_t m = a.x < a.y ? a.x : a.y, n = b.x < b.y ? b.x : b.y;
    return m < n ? m : n;
}

// The flush: one coalesced global atomic per touched pixel whose nearest key
// it lowers.
__device__ __forceinline__ void raster_wave_flush(uint64_t *__restrict__ fb, const uint64_t *w_tile,
                                                  MinFlush &f, bool l2 = false)
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t base = lds_addr(w_tile);
    gu64 *gfb = global_ptr(fb);
    arrive(f.cur);
    if (f.t.area == 0)
        return;
    if (lane < f.t.area) {
        const uint64_t v = tile_nearest(base, lane, f.four);
        if (v < f.cur)
            __hip_atomic_fetch_min(gfb + f.p0, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    for (uint32_t i = lane + 64; i < f.t.area; i += 64) {
        const uint64_t v = tile_nearest(base, i, f.four);
        if (v != ~0ull) {
            gu64 *dst = gfb + tile_pixel(f.t, i);
            const uint64_t was = read_nearest(dst, l2);
            if (v < was)
                __hip_atomic_fetch_min(dst, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    wave_sync();   // the tile is free for the next use
}

// Key of a point of any wave; clears `in` for a point that takes no part.
template <bool PW, int ZK>
__device__ __forceinline__ uint64_t key_any(const Proj &P, const Trans &T, float x, float y,
                                            float z, uint32_t c, bool &in)
{
    own(x), own(y), own(z);   // nothing of ChunkKey's is kept for here
    float cw = 0.0f, iw = 0.0f;
    if constexpr (ZK != 0) {
        cw = clip_w(P, T, x, y, z);
        if constexpr (ZK == RZ_DEPTH_GL24)
            iw = recip_rn(cw);
    }
    const uint64_t q = depth_enc<PW, ZK>(P, T, x, y, z, cw, iw, in);
    return (q << 24) | ((uint64_t)c & kRgbMask);
}

// A wave's points on screen: the first half of its depth pass.
template <int PPT>
struct WaveView {
    float fx[PPT], fy[PPT];   // window positions
    Box box;                  // of the on-screen points
    Where where;
    uint32_t behind;          // as sort_w leaves it
};

// False when the wave has nothing left to do: no point on screen, or points whose w
// needs the IEEE quotient, which go to the framebuffer one by one here.
template <int PPT, bool PW, int ZK>
__device__ __forceinline__ bool wave_view(const Proj &P, const Trans &T, uint64_t *__restrict__ fb,
                                          const float (&x)[PPT], const float (&y)[PPT],
                                          const float (&z)[PPT], const uint32_t (&c)[PPT],
                                          WaveView<PPT> &v)
{
    v.behind = 0u;
    v.where = window_all<PPT>(P, T, x, y, z, v.fx, v.fy, v.box);
    if (v.where == kOffScreen)
        return false;
    if (v.where == kMixed && sort_w<PPT>(P, T, x, y, z, v.behind)) {   // no wave in practice
        gu64 *gfb = global_ptr(fb);
#pragma unroll
        for (int j = 0; j < PPT; ++j) {
            float xx = x[j], yy = y[j], zz = z[j];
            own(xx), own(yy), own(zz);
            uint32_t px, py;
            uint64_t q;
            if (fragment_enc<PW, ZK>(P, T, xx, yy, zz, px, py, q))
                __hip_atomic_fetch_min(gfb + (__umul24(py, (uint32_t)P.width) + px),
                                       (q << 24) | ((uint64_t)c[j] & kRgbMask), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
            __builtin_amdgcn_sched_barrier(0);
        }
        return false;
    }
    if (v.where != kOnScreen) {
        v.box = window_box<PPT>(P, v.fx, v.fy, v.behind);
        return v.box.x1 <= kMaxPixel;   // some point on screen
    }
    return true;
}

// The second half of a wave that spreads too far for its tile: groups of four points.
// Consecutive points of a thread in one pixel send one atomic, and (AHEAD) a group's
// early-out reads are sent before the atomics of the group before it, which they would
// have to wait for otherwise (one counter covers all memory operations of a wave, in
// order).
template <int PPT, bool PW, int ZK, bool AHEAD>
__device__ __forceinline__ void raster_spread(const Proj &P, const Trans &T,
                                              uint64_t *__restrict__ fb, const float (&x)[PPT],
                                              const float (&y)[PPT], const float (&z)[PPT],
                                              const uint32_t (&c)[PPT], const WaveView<PPT> &v,
                                              bool early)
{
    gu64 *gfb = global_ptr(fb);
    const uint32_t width = (uint32_t)P.width;
    const ChunkKey<PW, ZK> key_of(P, T, x[0], y[0], z[0]);
    constexpr int G = 4, N = PPT / G;
    uint32_t pix[2][G];
    uint64_t key[2][G], cur[2][G];
    bool live[2][G];
    bool general = !PW;   // keys of points in any range
    auto read = [&](int g) {
        const int b = g & 1;
        bool vis[G], run = false;
#pragma unroll
        for (int k = 0; k < G; ++k) {
            const int j = G * g + k;
            float wx = v.fx[j], wy = v.fy[j];
            own(wx), own(wy);
            vis[k] = visible(P, wx, wy, v.behind, j);
            pix[b][k] = __umul24((uint32_t)(int32_t)(vis[k] ? wy : 0.0f), width) +
                        (uint32_t)(int32_t)(vis[k] ? wx : 0.0f);
        }
        if (!general) {
            bool all = true;
#pragma unroll
            for (int k = 0; k < G; ++k) {
                const int j = G * g + k;
                live[b][k] = true;
                key[b][k] = key_of(x[j], y[j], z[j], c[j], live[b][k]);
                all = all & (live[b][k] | !vis[k]);
                live[b][k] = live[b][k] & vis[k];
            }
            general = wave_any(!all);   // and so for the groups after it
        }
        if (general) {
#pragma unroll
            for (int k = 0; k < G; ++k) {
                const int j = G * g + k;
                live[b][k] = vis[k];
                key[b][k] = key_any<PW, ZK>(P, T, x[j], y[j], z[j], c[j], live[b][k]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int k = 1; k < G; ++k)
            run = run | (live[b][k] & live[b][k - 1] & (pix[b][k] == pix[b][k - 1]));
        if (wave_any(run)) {
#pragma unroll
            for (int k = 1; k < G; ++k) {
                const bool same = live[b][k] & live[b][k - 1] & (pix[b][k] == pix[b][k - 1]);
                const uint64_t lo = key[b][k] < key[b][k - 1] ? key[b][k] : key[b][k - 1];
                key[b][k] = same ? lo : key[b][k];
                live[b][k - 1] = live[b][k - 1] & !same;
            }
        }
#pragma unroll
        for (int k = 0; k < G; ++k)   // a point that takes no part reads pixel 0
            cur[b][k] = early ? read_nearest(gfb + (live[b][k] ? pix[b][k] : 0u), false) : ~0ull;
        __builtin_amdgcn_sched_barrier(0);
    };
    if (AHEAD)
        read(0);
#pragma unroll
    for (int g = 0; g < N; ++g) {
        const int b = g & 1;
        if (!AHEAD)
            read(g);
        else if (g + 1 < N)
            read(g + 1);
#pragma unroll
        for (int k = 0; k < G; ++k)
            if (live[b][k] & (key[b][k] < cur[b][k]))
                __hip_atomic_fetch_min(gfb + pix[b][k], key[b][k], __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The second half, in the wave's own tile where its rectangle fits (raster_chunk_wave).
template <int PPT, bool PW, int ZK, bool AHEAD>
__device__ __forceinline__ void raster_view(const Proj &P, const Trans &T,
                                            uint64_t *__restrict__ fb, const float (&x)[PPT],
                                            const float (&y)[PPT], const float (&z)[PPT],
                                            const uint32_t (&c)[PPT], const WaveView<PPT> &v,
                                            uint64_t *w_tile, uint32_t words, MinFlush &flush,
                                            bool l2, bool early)
{
    gu64 *gfb = global_ptr(fb);
    const uint32_t lane = threadIdx.x & 63u;
    const WaveTile t = wave_tile(P, v.box);
    const ChunkKey<PW, ZK> key_of(P, T, x[0], y[0], z[0]);
    if (t.area <= words) {
        const uint32_t base = lds_addr(w_tile);
        const uint32_t p0 = tile_pixel(t, lane);
        uint64_t cur = 0ull;
        if (lane < t.area)
            cur = read_nearest(gfb + p0, l2);
        const bool four = 4 * t.area <= words;
        const uint32_t sh = four ? 5u : 3u;
        const uint32_t bytes = t.area << sh;
        const uint32_t first = tile_first(t, base + (four ? 8 * (lane & 3u) : 0u), sh);
        auto clear = [&] {
            u64x2 none;
            none.x = none.y = ~0ull;
            if (16 * lane < bytes)
                *lds_ptr2(base + 16 * lane) = none;
            for (uint32_t i = 1024 + 16 * lane; i < bytes; i += 1024)
                *lds_ptr2(base + i) = none;
            wave_sync();
        };
        clear();
        bool in = v.where == kOnScreen;
        if (v.where == kOnScreen) {
#pragma unroll
            for (int j = 0; j < PPT; ++j) {
                __hip_atomic_fetch_min(lds_ptr(tile_entry(t, v.fx[j], v.fy[j], sh, first)),
                                       key_of(x[j], y[j], z[j], c[j], in), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
                if (j % 2)
                    __builtin_amdgcn_sched_barrier(0);
            }
            wave_sync();
        }
        if (wave_any(!in)) {   // flags per point
            clear();
#pragma unroll
            for (int j = 0; j < PPT; ++j) {
                float px = v.fx[j], py = v.fy[j];
                own(px), own(py);
                bool live = visible(P, px, py, v.behind, j);
                const uint64_t key = key_any<PW, ZK>(P, T, x[j], y[j], z[j], c[j], live);
                if (live)
                    __hip_atomic_fetch_min(lds_ptr(tile_entry(t, px, py, sh, first)), key,
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                __builtin_amdgcn_sched_barrier(0);
            }
            wave_sync();
        }
        flush = MinFlush{t, p0, cur, four};
        return;
    }
    raster_spread<PPT, PW, ZK, AHEAD>(P, T, fb, x, y, z, c, v, early);
}

// Depth pass over one chunk with a private LDS tile per wave: like
// raster_chunk with BIN, but every wave gathers its own 64 * PPT fragments
// in its own slice of `words` keys (w_tile), so no workgroup barrier is needed.
// Same result bits as raster_chunk, for any tile size.
// raster_wave_flush must follow with the same `flush`.  Without `early`, fragments
// of a wave that does not fit its tile go to the framebuffer unread.
//
// A wave whose points are all on screen and, as it turns out, in one range of
// the depth map and in [near, far) needs no flag per point, and neither the
// clamp nor the test for a slow reciprocal.  Every other wave goes on from the same
// window positions with flags per point (key_any), so that no point is loaded or
// projected again.
//
// The nearest keys that the flush compares with are read before the depths are
// computed, so that their latency passes meanwhile (a key read early is an upper
// bound of the later one).
//
// A tile that fits four times is kept four times, lane i taking copy i & 3:
// neighbouring lanes hold neighbouring points, and LDS atomics of one address
// follow each other one per cycle (a depth pass of 100M points over 8 views:
// 1.99 ms with one copy, 45% of it in such conflicts, 1.50 ms with four).
template <int PPT, bool PW, int ZK = 0, bool AHEAD = true>
__device__ __forceinline__ void raster_chunk_wave(const Proj &P, const Trans &T,
                                                  uint64_t *__restrict__ fb,
                                                  const float (&x)[PPT], const float (&y)[PPT],
                                                  const float (&z)[PPT], const uint32_t (&c)[PPT],
                                                  uint64_t *w_tile, uint32_t words,
                                                  MinFlush &flush, bool l2 = false,
                                                  bool early = true)
{
    WaveView<PPT> v;
    flush.t.area = 0;
    flush.cur = 0;
    if (wave_view<PPT, PW, ZK>(P, T, fb, x, y, z, c, v))
        raster_view<PPT, PW, ZK, AHEAD>(P, T, fb, x, y, z, c, v, w_tile, words, flush, l2, early);
}

// raster_chunk_wave for the kGroupWaves waves of one workgroup, with
// one tile in place of theirs where they cover the same pixels: the rectangle of all
// takes at most half of theirs together and fits their tiles' words.  That is an
// unordered cloud on few pixels, where every wave has an atomic for every pixel, and
// atomics of one pixel follow each other (about 27 ns each): the smaller the waves,
// the more of them.  Frames of 700k points on spheres in random order, waves of 256
// points alone / with this / waves of 1024 points: on 24 x 24 pixels 80.9 / 24.8 / 32.3
// us, on 32 x 32 204 / 29.8 / 30.1, at 1280x720 from so far away that they cover about
// 27 x 27 pixels 151 / 36.6 / 39.4; 2M points there 408 / 60.0 / 60.8.  What the barrier
// costs, depth passes at 640x480 without / with: spheres in random order 20k points 5.76 /
// 6.18 us, 100k 7.64 / 8.04, 300k 20.4 / 19.8, 1M 58.3 / 58.7, terrain 6.42 / 5.98, 7.00 /
// 7.44, 8.00 / 7.56, 7.32 / 7.20.  s_tiles: `words` keys of each wave, one wave after
// the other.
template <int PPT, bool PW, int ZK = 0>
__device__ __forceinline__ void raster_chunk_group(const Proj &P, const Trans &T,
                                                   uint64_t *__restrict__ fb,
                                                   const float (&x)[PPT], const float (&y)[PPT],
                                                   const float (&z)[PPT], const uint32_t (&c)[PPT],
                                                   uint64_t *s_tiles, uint32_t words,
                                                   uint32_t (*s_box)[4], MinFlush &flush,
                                                   bool early)
{
    WaveView<PPT> v;
    flush.t.area = 0;
    flush.cur = 0;
    const bool some = wave_view<PPT, PW, ZK>(P, T, fb, x, y, z, c, v);
    const uint32_t wave = threadIdx.x >> 6;
    const uint32_t limit = words * kGroupWaves;
    if ((threadIdx.x & 63u) == 0) {
        s_box[wave][0] = some ? v.box.x0 : ~0u;
        s_box[wave][1] = some ? v.box.y0 : ~0u;
        s_box[wave][2] = some ? v.box.x1 : 0u;
        s_box[wave][3] = some ? v.box.y1 : 0u;
    }
    // a wave beyond the shared tile by itself: its atomics need not wait for the others
    const bool alone = some && (v.box.x1 - v.box.x0 + 1) * (v.box.y1 - v.box.y0 + 1) > limit;
    if (alone)
        raster_spread<PPT, PW, ZK, true>(P, T, fb, x, y, z, c, v, early);
    __syncthreads();
    // lane i takes wave i & 3's rectangle; two steps over the quad make them one
    const uint32_t *w = s_box[threadIdx.x & (kGroupWaves - 1)];
    uint32_t x0 = w[0], y0 = w[1], x1 = w[2], y1 = w[3];
    // the sum of the areas, those beyond 2^16 pixels counted as that
    uint32_t sum = x0 > x1 ? 0u : min((x1 - x0 + 1) * (y1 - y0 + 1), 1u << 16);
    x0 = quad_min(x0), y0 = quad_min(y0), x1 = ~quad_min(~x1), y1 = ~quad_min(~y1);
    sum = quad_sum(sum);
    Box all;
    all.x0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)x0);
    all.y0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)y0);
    all.x1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)x1);
    all.y1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)y1);
    sum = (uint32_t)__builtin_amdgcn_readfirstlane((int)sum);
    const WaveTile t = wave_tile(P, all);
    if (t.area > limit || 2 * t.area > sum) {   // (nothing on screen: an area, no sum)
        if (some && !alone)
            raster_view<PPT, PW, ZK, true>(P, T, fb, x, y, z, c, v, s_tiles + wave * words, words,
                                           flush, false, early);
        return;
    }
    const uint32_t base = lds_addr(s_tiles);
    const bool four = 4 * t.area <= limit;
    const uint32_t sh = four ? 5u : 3u;
    const uint32_t first = tile_first(t, base + (four ? 8 * (threadIdx.x & 3u) : 0u), sh);
    for (uint32_t i = threadIdx.x; i < t.area << (sh - 3); i += blockDim.x)
        *lds_ptr(base + 8 * i) = ~0ull;
    __syncthreads();
    if (some) {
#pragma unroll
        for (int j = 0; j < PPT; ++j) {
            bool live = visible(P, v.fx[j], v.fy[j], v.behind, j);
            const uint64_t key = key_any<PW, ZK>(P, T, x[j], y[j], z[j], c[j], live);
            if (live)
                __hip_atomic_fetch_min(lds_ptr(tile_entry(t, v.fx[j], v.fy[j], sh, first)), key,
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
    __syncthreads();
    gu64 *gfb = global_ptr(fb);
    for (uint32_t i = threadIdx.x; i < t.area; i += blockDim.x) {
        const uint64_t m = tile_nearest(base, i, four);
        if (m != ~0ull) {
            gu64 *dst = gfb + tile_pixel(t, i);
            if (m < read_nearest(dst, false))
                __hip_atomic_fetch_min(dst, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// Accumulation pass of high-quality splatting over one chunk (section 2.2).
// Reprojects every point, compares its depth with the finished depth pass
// and, inside the eps window, adds its colour and a count:
//   acc[2p] += R + (G << 32),  acc[2p+1] += B + (1 << 32).
// As in the depth pass, consecutive accepted fragments of a thread in one
// pixel are summed in registers, and with BIN the workgroup's sums are
// gathered in an LDS tile (64-bit LDS adds) and flushed once per pixel.
// Integer sums are order independent, so every variant gives the same bits.
// PW: the piecewise depth map's window test (linear depths in double).
// Barrier rules as for raster_chunk.
template <int PPT, bool BIN, bool PW>
__device__ __forceinline__ void accum_chunk(const Proj &P, uint32_t eps_num, uint32_t eps_den,
                                            const uint64_t *__restrict__ fb,
                                            uint64_t *__restrict__ acc,
                                            const float (&x)[PPT], const float (&y)[PPT],
                                            const float (&z)[PPT], const uint32_t (&c)[PPT],
                                            const bool (&in)[PPT], uint64_t *s_tile,
                                            uint32_t (*s_box)[4])
{
    uint32_t px[PPT], py[PPT], pix[PPT];
    uint64_t q[PPT];
    bool ok[PPT];
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
        uint32_t a = 0, b = 0;
        uint64_t qq = 0;
        ok[j] = fragment<PW>(P, x[j], y[j], z[j], a, b, qq) & in[j];
        px[j] = a;
        py[j] = b;
        pix[j] = __umul24(b, (uint32_t)P.width) + a;   // both below 2^15
        q[j] = qq;
    }
    // eps window against the finished depth pass: all loads first
    // (discarded fragments read pixel 0, always in bounds), then the tests
    uint64_t fbv[PPT];
#pragma unroll
    for (int j = 0; j < PPT; ++j)
        fbv[j] = fb[ok[j] ? pix[j] : 0u];
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
        const uint64_t qmin = fbv[j] >> 24;
        ok[j] = in_window_live<PW>(P, eps_num, eps_den, q[j], qmin, ok[j]);
    }
    uint64_t w0[PPT], w1[PPT];
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
        w0[j] = (uint64_t)(c[j] & 0xFFu) | ((uint64_t)((c[j] >> 8) & 0xFFu) << 32);
        w1[j] = (uint64_t)((c[j] >> 16) & 0xFFu) | (1ull << 32);
    }
#pragma unroll
    for (int j = 1; j < PPT; ++j) {
        const bool same = ok[j] && ok[j - 1] && pix[j] == pix[j - 1];
        w0[j] += same ? w0[j - 1] : 0ull;
        w1[j] += same ? w1[j - 1] : 0ull;
        ok[j - 1] = ok[j - 1] && !same;
    }

    bool direct[PPT];
    Box box{1, 1, 0, 0};
    uint32_t bw = 0, bh = 0;
    bool tiled = false;
    if (BIN) {
        box = block_box<PPT>(px, py, ok, s_box);
        if (box.x0 <= box.x1) {
            bw = box.x1 - box.x0 + 1;
            bh = box.y1 - box.y0 + 1;
            tiled = (uint64_t)bw * bh <= kTileHq;
        }
    }
    if (tiled) {
        const uint32_t area = bw * bh;
        for (uint32_t i = threadIdx.x; i < 2 * area; i += blockDim.x)
            s_tile[i] = 0ull;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < PPT; ++j) {
            const uint32_t tx = px[j] - box.x0, ty = py[j] - box.y0;
            const bool inside = ok[j] && tx < bw && ty < bh;
            direct[j] = ok[j] && !inside;
            if (inside) {
                uint64_t *t = &s_tile[2 * (ty * bw + tx)];
                __hip_atomic_fetch_add(t, w0[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                __hip_atomic_fetch_add(t + 1, w1[j], __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < area; i += blockDim.x) {
            const uint64_t a1 = s_tile[2 * i + 1];
            if (a1 != 0ull) {
                const uint64_t a0 = s_tile[2 * i];
                const uint32_t r = i / bw;
                const uint32_t col = i - r * bw;
                uint64_t *dst =
                    acc + 2 * (uint64_t)(__umul24(box.y0 + r, (uint32_t)P.width) + box.x0 + col);
                __hip_atomic_fetch_add(dst, a0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_fetch_add(dst + 1, a1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    } else {
#pragma unroll
        for (int j = 0; j < PPT; ++j)
            direct[j] = ok[j];
    }
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
        if (direct[j]) {
            uint64_t *a = acc + 2 * (uint64_t)pix[j];
            __hip_atomic_fetch_add(a, w0[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_fetch_add(a + 1, w1[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// Adds the sums a0, a1 to pixel p of the accumulator.
__device__ __forceinline__ void add_pixel(gu64 *acc, uint32_t p, uint64_t a0, uint64_t a1)
{
    gu64 *dst = acc + 2 * (uint64_t)p;
    __hip_atomic_fetch_add(dst, a0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_add(dst + 1, a1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Splat sums of up to 512 points in one word, R | G << 17 | B << 34 | count << 51: no
// field can carry into the next (512 * 255 < 2^17, 512 < 2^13).
__device__ __forceinline__ uint64_t pack_sums(uint32_t c)
{
    const uint32_t r = c & 0xFFu, g = (c >> 8) & 0xFFu, b = (c >> 16) & 0xFFu;
    return ((uint64_t)((b << 2) | (1u << 19)) << 32) | (r | (g << 17));
}

// The accumulator's two words of them.
__device__ __forceinline__ uint64_t sums_rg(uint64_t w)
{
    return (w & 0x1FFFFull) | (((w >> 17) & 0x1FFFFull) << 32);
}
__device__ __forceinline__ uint64_t sums_bn(uint64_t w)
{
    return ((w >> 34) & 0x1FFFFull) | ((w >> 51) << 32);
}

// The second half of a wave's accumulate pass with flags per point: waves that
// accum_wave_fast does not take.  Consecutive points of a thread in one pixel are summed
// in registers.  A wave of at most 512 points (PPT <= 8) keeps its sums in its tile as
// packed words, larger waves as the accumulator's own two words.
template <int PPT, bool PW>
__device__ __forceinline__ void accum_view(const Proj &P, const Trans &T, const Eps &eps,
                                           const uint64_t *__restrict__ fb,
                                           uint64_t *__restrict__ acc, const float (&x)[PPT],
                                           const float (&y)[PPT], const float (&z)[PPT],
                                           const uint32_t (&c)[PPT], const float (&fx)[PPT],
                                           const float (&fy)[PPT], uint32_t behind, const Box &box,
                                           uint64_t *w_tile, uint32_t words)
{
    constexpr bool kPacked = PPT <= 8;
    constexpr uint32_t kSh = kPacked ? 3u : 4u;   // bytes per pixel, log2
    const uint32_t lane = threadIdx.x & 63u;
    const WaveTile t = wave_tile(P, box);
    const bool tiled = tile_fits(t.area, words, kSh);
    const uint32_t base = lds_addr(w_tile);
    const gu64 *gfb = (const gu64 *)global_ptr(fb);
    gu64 *gacc = global_ptr(acc);
    if (tiled) {
        for (uint32_t i = lane; i < (t.area << (kSh - 3)); i += 64)
            *lds_ptr(base + 8 * i) = 0ull;
        wave_sync();
    }
    const uint32_t first = tile_first(t, base, kSh);
    // groups of four points, the nearest depths of the next one in flight
    constexpr int G = 4, N = PPT / G;
    uint32_t at[2][G];   // LDS address of the pixel's entry, or the pixel beside a tile
    uint64_t q[2][G], near[2][G];
    bool ok[2][G];
    auto read = [&](int g) {
        const int b = g & 1;
#pragma unroll
        for (int k = 0; k < G; ++k) {
            const int j = G * g + k;
            float wx = fx[j], wy = fy[j];
            own(wx), own(wy);
            ok[b][k] = visible(P, wx, wy, behind, j);
            const uint32_t px = (uint32_t)(int32_t)(ok[b][k] ? wx : 0.0f);
            const uint32_t py = (uint32_t)(int32_t)(ok[b][k] ? wy : 0.0f);
            float xx = x[j], yy = y[j], zz = z[j];
            own(xx), own(yy), own(zz);
            q[b][k] = depth_enc<PW, 0>(P, T, xx, yy, zz, 0.0f, 0.0f, ok[b][k]);
            const uint32_t pix = __umul24(py, t.width) + px;
            // a discarded fragment reads pixel 0
            near[b][k] = gfb[ok[b][k] ? pix : 0u];
            at[b][k] = tiled ? ((__umul24(py, t.bw) + px) << kSh) + first : pix;
            own(at[b][k]);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    read(0);
#pragma unroll
    for (int g = 0; g < N; ++g) {
        const int b = g & 1;
        if (g + 1 < N)
            read(g + 1);
        uint64_t sum[G];
        bool in[G], run = false;
#pragma unroll
        for (int k = 0; k < G; ++k) {
            in[k] = in_window_live<PW>(P, eps.num, eps.den, q[b][k], near[b][k] >> 24, ok[b][k]);
            sum[k] = pack_sums(c[G * g + k]);
            if (k > 0)
                run = run | (in[k] & in[k - 1] & (at[b][k] == at[b][k - 1]));
        }
        if (wave_any(run)) {
#pragma unroll
            for (int k = 1; k < G; ++k) {
                const bool same = in[k] & in[k - 1] & (at[b][k] == at[b][k - 1]);
                sum[k] += same ? sum[k - 1] : 0ull;
                in[k - 1] = in[k - 1] & !same;
            }
        }
#pragma unroll
        for (int k = 0; k < G; ++k) {
            if (!in[k])
                continue;
            if (!tiled) {
                add_pixel(gacc, at[b][k], sums_rg(sum[k]), sums_bn(sum[k]));
            } else if (kPacked) {
                __hip_atomic_fetch_add(lds_ptr(at[b][k]), sum[k], __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
            } else {
                __hip_atomic_fetch_add(lds_ptr(at[b][k]), sums_rg(sum[k]), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
                __hip_atomic_fetch_add(lds_ptr(at[b][k]) + 1, sums_bn(sum[k]), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    if (!tiled)
        return;
    wave_sync();
    for (uint32_t i = lane; i < t.area; i += 64) {
        const uint64_t w = *lds_ptr(base + (i << kSh));
        const uint64_t a0 = kPacked ? sums_rg(w) : w;
        const uint64_t a1 = kPacked ? sums_bn(w) : *lds_ptr(base + (i << kSh) + 8);
        if (a1 != 0ull)   // count > 0
            add_pixel(gacc, tile_pixel(t, i), a0, a1);
    }
    wave_sync();   // the tile is free for the next use
}

// What accum_chunk_wave leaves to be flushed: its tile (area 0: nothing) and the
// pixels of the lane's first entries.
template <int PPT>
struct SumFlush {
    static constexpr int kPre = PPT / 2;   // entries per lane whose depths are read ahead
    WaveTile t;
    uint32_t pix[kPre];
    bool four;
};

template <int PPT>
__device__ __forceinline__ void accum_wave_flush(uint64_t *__restrict__ acc, const uint64_t *w_tile,
                                                 const SumFlush<PPT> &f)
{
    if (f.t.area == 0)
        return;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t base = lds_addr(w_tile), sh = f.four ? 5u : 4u;
    gu64 *gacc = global_ptr(acc);
    auto flush = [&](uint32_t i, uint32_t p) {
        uint64_t a0 = 0, a1 = 0;
        auto add = [&](uint64_t w) {
            a0 += (w & 0xFFFFull) | (((w >> 16) & 0xFFFFull) << 32);
            a1 += ((w >> 32) & 0xFFFFull) | ((w >> 48) << 32);
        };
        const u64x2 a = *lds_ptr2(base + (i << sh));
        if (f.four) {   // pairs hold at most 256 points
            const u64x2 b = *lds_ptr2(base + (i << sh) + 16);
            add(a.x + a.y);
            add(b.x + b.y);
        } else {
            add(a.x);
            add(a.y);
        }
        if (a1 != 0ull) {   // count > 0
            own(p);   // its address is not made before
            add_pixel(gacc, p, a0, a1);
        }
    };
#pragma unroll
    for (int k = 0; k < SumFlush<PPT>::kPre; ++k) {
        if (k > 0 && f.t.area <= 64u * k)
            break;
        if (lane + 64 * k < f.t.area)
            flush(lane + 64 * k, f.pix[k]);
    }
    for (uint32_t i = lane + 64 * SumFlush<PPT>::kPre; i < f.t.area; i += 64)
        flush(i, tile_pixel(f.t, i));
    wave_sync();   // the tile is free for the next use
}

// The second half for a wave wholly on screen, under a map and a window of which the
// threshold of a pixel is known (window_threshold).
//
// The window test is one comparison per point against its pixel's threshold.  The
// thresholds lie in LDS beside the sums: the nearest depths of the rectangle are read in
// coalesced rows while the depths are computed, instead of one by one.
//
// Sums: R | G << 16 | B << 32 | count << 48 in copies of the tile, four where
// they fit, else two (neighbouring lanes hold neighbouring points, and the LDS
// adds of one address follow each other one per cycle).  One of two copies, or a
// pair of the four, takes the points of 32 lanes of at most 8 points:
// 256 * 255 < 2^16, so no field carries before the fields are unpacked.
template <int PPT>
__device__ __forceinline__ void accum_wave_fast(const Proj &P, const Trans &T, const Eps &eps,
                                                const uint64_t *__restrict__ fb,
                                                const float (&x)[PPT], const float (&y)[PPT],
                                                const float (&z)[PPT], const uint32_t (&c)[PPT],
                                                const float (&fx)[PPT], const float (&fy)[PPT],
                                                const Box &box, uint64_t *w_tile, uint32_t words,
                                                SumFlush<PPT> &flush)
{
    const uint32_t lane = threadIdx.x & 63u;
    const WaveTile t = wave_tile(P, box);
    const gu64 *gfb = (const gu64 *)global_ptr(fb);
    constexpr int kPre = SumFlush<PPT>::kPre;
    const uint32_t base = lds_addr(w_tile);
    const bool four = 5 * t.area <= words;
    const uint32_t sh = four ? 5u : 4u;
    const uint32_t thr = base + (t.area << sh);   // the thresholds' LDS address
    uint32_t pix[kPre] = {};
    uint64_t near[kPre];
#pragma unroll
    for (int k = 0; k < kPre; ++k) {
        if (k > 0 && t.area <= 64u * k)
            break;
        pix[k] = tile_pixel(t, lane + 64 * k);
        near[k] = lane + 64 * k < t.area ? gfb[pix[k]] : 0ull;
    }
    u64x2 zero;
    zero.x = zero.y = 0ull;
    for (uint32_t i = 16 * lane; i < (t.area << sh); i += 1024)
        *lds_ptr2(base + i) = zero;
    double q[PPT];   // infinite for a point out of range, beyond every threshold
#pragma unroll
    for (int g = 0; g < PPT; g += 4) {
        double d[4];
        bool out = false;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int j = g + k;
            d[k] = depth_of(P, T.td, x[j], y[j], z[j]);
            q[j] = floor((d[k] - P.o) * P.s);
            out = out | (d[k] < P.dlo[0]) | (d[k] >= P.dhi[0]);
            if (k % 2)
                __builtin_amdgcn_sched_barrier(0);
        }
        if (wave_any(out)) {   // (a NaN fails the window test anyway)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const bool in = (d[k] >= P.near_) & (d[k] < P.far_);
                q[g + k] = in ? fmin(q[g + k], kQMax) : __builtin_inf();
            }
        }
    }
#pragma unroll
    for (int j = 0; j < PPT; ++j)   // not before the depths are there
        asm volatile("" : "+v"(near[0]) : "v"(q[j]));
#pragma unroll
    for (int k = 1; k < kPre; ++k)
        if (t.area > 64u * k)
            arrive(near[k]);
    typedef __attribute__((address_space(3))) double lf64;
#pragma unroll
    for (int k = 0; k < kPre; ++k) {
        if (k > 0 && t.area <= 64u * k)
            break;
        if (lane + 64 * k < t.area)
            *(lf64 *)(uintptr_t)(thr + 8 * (lane + 64 * k)) = window_threshold(P, eps, near[k]);
    }
    for (uint32_t i = lane + 64 * kPre; i < t.area; i += 64)
        *(lf64 *)(uintptr_t)(thr + 8 * i) = window_threshold(P, eps, gfb[tile_pixel(t, i)]);
    wave_sync();
    const uint32_t sub = lane & (four ? 3u : 1u);
    const uint32_t first = tile_first(t, base + 8 * sub, sh);
    const uint32_t tfirst = tile_first(t, thr, 3);
    constexpr int G = 4;   // thresholds in flight
#pragma unroll
    for (int g = 0; g < PPT; g += G) {
        uint32_t e[G];
        double most[G];
#pragma unroll
        for (int k = 0; k < G; ++k) {
            e[k] = __umul24((uint32_t)(int32_t)fy[g + k], t.bw) +
                   (uint32_t)(int32_t)fx[g + k];
            most[k] = *(lf64 *)(uintptr_t)((e[k] << 3) + tfirst);
        }
#pragma unroll
        for (int k = 0; k < G; ++k) {
            if (q[g + k] <= most[k]) {
                const uint32_t lo = __builtin_amdgcn_perm(1u, c[g + k], 0x0c010c00u);   // R, G
                const uint32_t hi = __builtin_amdgcn_perm(1u, c[g + k], 0x0c040c02u);   // B, 1
                __hip_atomic_fetch_add(lds_ptr((e[k] << sh) + first),
                                       ((uint64_t)hi << 32) | lo, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
    }
    wave_sync();
    flush.t = t;
    flush.four = four;
#pragma unroll
    for (int k = 0; k < kPre; ++k)
        flush.pix[k] = pix[k];
}

// Accumulate pass over one chunk with a private LDS tile per wave of `words`
// words.  Same result bits as accum_chunk.  accum_wave_flush must follow with
// the same `flush`.
//
// As in the depth pass, a wave whose points are all on screen needs no flag per point
// (accum_wave_fast); every other one goes on from the same window positions with flags
// (accum_view), and so do waves whose rectangle does not fit the tile, piecewise maps,
// and windows whose products are not exact in double precision.
template <int PPT, bool PW>
__device__ __forceinline__ void accum_chunk_wave(const Proj &P, const Trans &T, const Eps &eps,
                                                 const uint64_t *__restrict__ fb,
                                                 uint64_t *__restrict__ acc, const float (&x)[PPT],
                                                 const float (&y)[PPT], const float (&z)[PPT],
                                                 const uint32_t (&c)[PPT], uint64_t *w_tile,
                                                 uint32_t words, SumFlush<PPT> &flush)
{
    float fx[PPT], fy[PPT];
    Box box;
    uint32_t behind = 0u;
    flush.t.area = 0;
    const Where where = window_all<PPT>(P, T, x, y, z, fx, fy, box);
    if (where == kOffScreen)
        return;
    if (where == kMixed && sort_w<PPT>(P, T, x, y, z, behind)) {   // no wave in practice
#pragma unroll
        for (int j = 0; j < PPT; ++j) {
            float xx = x[j], yy = y[j], zz = z[j];
            own(xx), own(yy), own(zz);
            uint32_t px, py;
            uint64_t q;
            const bool live = fragment<PW>(P, T, xx, yy, zz, px, py, q);
            const uint32_t pix = __umul24(py, (uint32_t)P.width) + px;
            const uint64_t qmin = global_ptr(fb)[live ? pix : 0u] >> 24;
            if (in_window_live<PW>(P, eps.num, eps.den, q, qmin, live)) {
                const uint64_t w = pack_sums(c[j]);
                add_pixel(global_ptr(acc), pix, sums_rg(w), sums_bn(w));
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        return;
    }
    if (where != kOnScreen) {
        box = window_box<PPT>(P, fx, fy, behind);
        if (box.x1 > kMaxPixel)   // no point on screen
            return;
    }
    if constexpr (PPT <= 8) {   // the sums' 16-bit fields
        if (where == kOnScreen && !(PW && P.nr != 0) && window_exact(P, eps) &&
            3 * (box.x1 - box.x0 + 1) * (box.y1 - box.y0 + 1) <= words) {
            accum_wave_fast<PPT>(P, T, eps, fb, x, y, z, c, fx, fy, box, w_tile, words, flush);
            return;
        }
    }
    accum_view<PPT, PW>(P, T, eps, fb, acc, x, y, z, c, fx, fy, behind, box, w_tile, words);
}

// Colour of one pixel from its packed splat sums (section 2.2, third pass):
// per channel (2 * sum + count) / (2 * count), or the background.
__device__ __forceinline__ uint32_t hq_colour(uint64_t w0, uint64_t w1, uint32_t bg,
                                              bool &overflow)
{
    const uint64_t cnt = w1 >> 32;
    if (cnt == 0)
        return bg;
    overflow = cnt > kHqCountMax;
    const double den = 2.0 * (double)cnt;
    // numerators < 2^34: the double quotient floors exactly
    const uint32_t r = (uint32_t)floor((2.0 * (double)(w0 & 0xFFFFFFFFull) + (double)cnt) / den);
    const uint32_t g = (uint32_t)floor((2.0 * (double)(w0 >> 32) + (double)cnt) / den);
    const uint32_t b = (uint32_t)floor((2.0 * (double)(w1 & 0xFFFFFFFFull) + (double)cnt) / den);
    return (r & 0xFFu) | ((g & 0xFFu) << 8) | ((b & 0xFFu) << 16);
}

}  // namespace dev
}  // namespace rz
