// Points larger than one pixel and the float depth encodings (declared in
// include/rz.h, rasterize_points).  A point of size k covers the k x k pixels
// px - r .. px - r + k - 1 (r = (k - 1) / 2) around its own pixel, clipped to
// the screen: k^2 fragments with one key in the depth pass (section 2.1), and
// in the splat pass (section 2.2) every covered pixel tests the point
// against its own nearest depth.
//
// A wave of spatially ordered points does not make these fragments one by one.
// A covered pixel's nearest key is the minimum over the k x k centres that cover
// it, so the depth pass takes one LDS minimum per point, at its centre, and
// dilates the tile of centres when it is flushed, rows first, then columns.  In
// the splat pass a point inside the windows of all its covered pixels (nearly all
// are) adds its colour once, at its centre, and the flush sums the centres that
// cover each pixel, again rows first; a point outside all of them adds nothing;
// only the others test and add pixel by pixel.  The depth pass of 50M points at
// 1920x1080, k = 3: 360 us with k^2 minima per point, 190 us; the splat pass:
// 895 us, 280 us.  Waves that spread too far, or are not wholly on screen, take
// their covered pixels one by one.
//
// The nearest keys that a depth pass compares with are read through the XCD's L2
// (read_nearest): tiles of neighbouring waves overlap by k - 1 pixels, so the lines
// are met again.  Frames at 1920x1080, read past it / through it: 50M points, k = 2,
// 3, 5, 8, 16: 197 / 191, 196 / 188, 230 / 210, 530 / 417, 1273 / 978 us; 5M points
// 45 / 44, 54 / 54, 78 / 78, 150 / 150, 684 / 678; 0.5M (few waves fit their tile)
// 64 / 61, 111 / 108, 233 / 224, 444 / 428, 1281 / 1242.  Beside the tile that holds for
// sparse clouds only: 2M points with a stray one in 256, k = 2 and 3, 101 / 115 and 177 /
// 193 us, so waves with runs of points in one pixel read past it there.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rz.h"
#include "rz_device.h"
#include "rz_internal.h"
#include "rz_trace.h"

namespace rz {
namespace {

using namespace dev;

constexpr int kGenBlock = 256;
constexpr int kGenPpt = 4;   // one 16-byte group of points per thread
// LDS of a wave: 8 KiB, in the splat pass 16 KiB for squares above 5 pixels, whose
// covered rectangles are far larger than the rectangles of their centres.
constexpr uint32_t kHqWordsLarge = 2 * kWaveTileWords;
// Packed sums, R | G << 16 | B << 32 | count << 48.  A wave holds 64 * kGenPpt = 256
// points, and a point adds to a pixel at most once, so a pixel's count stays
// <= 256 and its channel sums <= 255 * 256 < 2^16: no field carries.
static_assert(64 * kGenPpt * 255 < (1 << 16), "packed sums");

// Covered pixels [lo, hi) along one axis for a point of size k at pixel c.
__device__ __forceinline__ void cover(uint32_t c, int32_t k, int32_t size, int32_t &lo,
                                      int32_t &hi)
{
    const int32_t a = (int32_t)c - (k - 1) / 2;
    lo = a < 0 ? 0 : a;
    hi = a + k > size ? size : a + k;
}

// Rectangle covered by the squares of a wave's points (centres in box),
// clipped to the screen; tiled when it fits `limit` pixels.
struct Cover {
    int32_t x0, y0;
    uint32_t bw, bh;
    bool tiled;
};

__device__ __forceinline__ Cover wave_cover(const Box &box, int32_t k, int32_t width,
                                            int32_t height, uint32_t limit)
{
    Cover c{0, 0, 0, 0, false};
    if (box.x0 > box.x1)
        return c;
    const int32_t r = (k - 1) / 2;
    const int32_t x0 = (int32_t)box.x0 - r, y0 = (int32_t)box.y0 - r;
    const int32_t x1 = (int32_t)box.x1 - r + k - 1, y1 = (int32_t)box.y1 - r + k - 1;
    c.x0 = x0 < 0 ? 0 : x0;
    c.y0 = y0 < 0 ? 0 : y0;
    const int32_t cx1 = x1 > width - 1 ? width - 1 : x1;
    const int32_t cy1 = y1 > height - 1 ? height - 1 : y1;
    c.bw = (uint32_t)(cx1 - c.x0 + 1);
    c.bh = (uint32_t)(cy1 - c.y0 + 1);
    c.tiled = (uint64_t)c.bw * c.bh <= limit;
    return c;
}

// The rectangle covered by the squares of the centres in a tile.
struct Covered {
    uint32_t x0, y0, w, h, area;
    float inv_w;
};

__device__ __forceinline__ Covered covered_rect(const Proj &P, const Box &box, int32_t k)
{
    const int32_t r = (k - 1) / 2;
    const int32_t x0 = max((int32_t)box.x0 - r, 0), y0 = max((int32_t)box.y0 - r, 0);
    const int32_t x1 = min((int32_t)box.x1 - r + k, P.width);
    const int32_t y1 = min((int32_t)box.y1 - r + k, P.height);
    Covered c;
    c.x0 = (uint32_t)x0;
    c.y0 = (uint32_t)y0;
    c.w = (uint32_t)(x1 - x0);
    c.h = (uint32_t)(y1 - y0);
    c.area = c.w * c.h;
    c.inv_w = __builtin_amdgcn_rcpf((float)c.w);   // tile_rc corrects it
    return c;
}

// f(k), with the usual sizes as compile-time constants.
template <int K>
struct Const {
    __device__ constexpr operator int() const { return K; }
};
template <typename F>
__device__ __forceinline__ void with_size(int32_t k, const F &f)
{
    switch (k) {
    case 2: f(Const<2>{}); break;
    case 3: f(Const<3>{}); break;
    case 4: f(Const<4>{}); break;
    case 5: f(Const<5>{}); break;
    default: f(k); break;
    }
}

// Column (or row) of the tile of centres that lies d before the last centre
// covering position p, kept inside [0, n): o = position 0 minus centre 0.
__device__ __forceinline__ uint32_t centre(uint32_t p, int32_t o, int32_t r, int32_t d, uint32_t n)
{
    const int32_t i = (int32_t)p + o + r - d;
    return (uint32_t)min(max(i, 0), (int32_t)n - 1);
}

// Flush of the depth pass: the tile of centres (t, `copies` keys per pixel at LDS
// address base) dilated by k x k into fb.  The rows' minima go to LDS behind the
// tile where they fit (`rows` then), else each pixel takes k^2 reads.
__device__ __forceinline__ void dilate_flush(const WaveTile &t, const Covered &v, int32_t k,
                                             uint32_t base, bool four, bool rows, gu64 *fb,
                                             uint64_t cur0)
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t bh = t.area / t.bw;   // uniform
    const int32_t r = (k - 1) / 2;
    const int32_t ox = (int32_t)v.x0 - (int32_t)t.x0, oy = (int32_t)v.y0 - (int32_t)t.y0;
    auto min_of = [](uint64_t a, uint64_t b) { return b < a ? b : a; };
    if (four) {   // one copy, in place of the first
        for (uint32_t i = lane; i < t.area; i += 64) {
            const u64x2 a = *lds_ptr2(base + 32 * i), b = *lds_ptr2(base + 32 * i + 16);
            *lds_ptr(base + 32 * i) = min_of(min_of(a.x, a.y), min_of(b.x, b.y));
        }
        wave_sync();
    }
    const uint32_t sh = four ? 5u : 3u;
    const uint32_t line = base + (t.area << sh);   // minima over rows: v.w columns, bh rows
    if (rows) {
        with_size(k, [&](auto kk) {
            for (uint32_t i = lane; i < v.w * bh; i += 64) {
                uint32_t row, col;
                tile_rc(i, v.w, v.inv_w, row, col);
                const uint32_t at = base + ((row * t.bw) << sh);
                uint64_t m = ~0ull;
                for (int d = 0; d < kk; ++d)
                    m = min_of(m, *lds_ptr(at + (centre(col, ox, r, d, t.bw) << sh)));
                *lds_ptr(line + 8 * i) = m;
            }
        });
        wave_sync();
    }
    for (uint32_t i = lane; i < v.area; i += 64) {
        uint32_t row, col;
        tile_rc(i, v.w, v.inv_w, row, col);
        uint64_t m = ~0ull;
        if (rows) {
            with_size(k, [&](auto kk) {
                for (int d = 0; d < kk; ++d)
                    m = min_of(m, *lds_ptr(line + 8 * (centre(row, oy, r, d, bh) * v.w + col)));
            });
        } else {
            for (int dy = 0; dy < k; ++dy) {
                const uint32_t at = base + ((centre(row, oy, r, dy, bh) * t.bw) << sh);
                for (int dx = 0; dx < k; ++dx)
                    m = min_of(m, *lds_ptr(at + (centre(col, ox, r, dx, t.bw) << sh)));
            }
        }
        if (m != ~0ull) {
            gu64 *dst = fb + (__umul24(v.y0 + row, t.width) + v.x0 + col);
            const uint64_t was = i == lane ? cur0 : read_nearest(dst, true);
            if (m < was)
                __hip_atomic_fetch_min(dst, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    wave_sync();
}

// Depth pass.  PW: piecewise maps; ZK: 0 for the integer maps, else the float
// encoding.
template <bool PW, int ZK>
__global__ void __launch_bounds__(kGenBlock) k_raster_points(Pts p, Proj P, int32_t k,
                                                             uint64_t *__restrict__ fb)
{
    extern __shared__ uint64_t s_waves[];
    uint64_t *w_tile = s_waves + (threadIdx.x >> 6) * kWaveTileWords;
    const int64_t chunk = (int64_t)blockIdx.x * kGenBlock * kGenPpt;
    float x[kGenPpt], y[kGenPpt], z[kGenPpt];
    uint32_t c[kGenPpt];
    load_points_nan<kGenPpt>(p, chunk, x, y, z, c);
    const uint32_t lane = threadIdx.x & 63u;
    const Trans T = lane_trans(P);
    const uint32_t base = lds_addr(w_tile);
    gu64 *gfb = global_ptr(fb);
    float fx[kGenPpt], fy[kGenPpt];
    Box box;
    const Where where = window_all<kGenPpt>(P, T, x, y, z, fx, fy, box);
    if (where == kOffScreen)
        return;
    if (where == kOnScreen) {
        const WaveTile t = wave_tile(P, box);
        if (t.area <= kWaveTileWords) {
            const Covered v = covered_rect(P, box, k);
            const uint32_t nrow = v.w * (t.area / t.bw);
            const bool four = 4 * t.area + nrow <= kWaveTileWords;
            const bool rows = four || t.area + nrow <= kWaveTileWords;
            uint64_t cur = 0ull;
            if (lane < v.area) {
                uint32_t row, col;
                tile_rc(lane, v.w, v.inv_w, row, col);
                cur = read_nearest(gfb + (__umul24(v.y0 + row, t.width) + v.x0 + col), true);
            }
            const uint32_t sh = four ? 5u : 3u;
            u64x2 none;
            none.x = none.y = ~0ull;
            for (uint32_t i = 16 * lane; i < (t.area << sh); i += 1024)
                *lds_ptr2(base + i) = none;
            wave_sync();
            const uint32_t first = tile_first(t, base + (four ? 8 * (lane & 3u) : 0u), sh);
            const ChunkKey<PW, ZK> key_of(P, T, x[0], y[0], z[0]);
            bool in = true;
#pragma unroll
            for (int j = 0; j < kGenPpt; ++j)
                __hip_atomic_fetch_min(lds_ptr(tile_entry(t, fx[j], fy[j], sh, first)),
                                       key_of(x[j], y[j], z[j], c[j], in), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
            wave_sync();
            arrive(cur);
            if (!wave_any(!in)) {
                dilate_flush(t, v, k, base, four, rows, gfb, cur);
                return;
            }
        }
    }
    // any other wave: flags per point, the squares pixel by pixel
    uint32_t px[kGenPpt], py[kGenPpt];
    uint64_t key[kGenPpt];
    bool live[kGenPpt];
#pragma unroll
    for (int j = 0; j < kGenPpt; ++j) {
        uint32_t a = 0, b = 0;
        uint64_t q = 0;
        live[j] = fragment_enc<PW, ZK>(P, T, x[j], y[j], z[j], a, b, q);
        px[j] = a;
        py[j] = b;
        key[j] = (q << 24) | ((uint64_t)c[j] & kRgbMask);
    }
    // consecutive points of a thread with one centre pixel cover the same
    // square: keep only their smaller key (k^2 atomics saved per merge)
    bool run = false;
#pragma unroll
    for (int j = 1; j < kGenPpt; ++j) {
        const bool same = live[j] && live[j - 1] && px[j] == px[j - 1] && py[j] == py[j - 1];
        const uint64_t lo = key[j] < key[j - 1] ? key[j] : key[j - 1];
        key[j] = same ? lo : key[j];
        live[j - 1] = live[j - 1] && !same;
        run = run | same;
    }
    // Waves with such runs are those of a dense ordered cloud with a stray point in them:
    // their neighbours lower the same pixels, and an older key costs an atomic.
    const bool l2 = __builtin_popcountll(__builtin_amdgcn_ballot_w64(run)) < 8;
    const Cover cv = wave_cover(wave_box<kGenPpt>(px, py, live), k, P.width, P.height,
                                kWaveTileMin);
    if (cv.tiled) {
        const uint32_t area = cv.bw * cv.bh;
        for (uint32_t i = lane; i < area; i += 64)
            w_tile[i] = ~0ull;
        wave_sync();
#pragma unroll
        for (int j = 0; j < kGenPpt; ++j) {
            if (!live[j])
                continue;
            int32_t x0, x1, y0, y1;
            cover(px[j], k, P.width, x0, x1);
            cover(py[j], k, P.height, y0, y1);
            for (int32_t yy = y0; yy < y1; ++yy)
                for (int32_t xx = x0; xx < x1; ++xx)
                    __hip_atomic_fetch_min(&w_tile[(uint32_t)(yy - cv.y0) * cv.bw +
                                                   (uint32_t)(xx - cv.x0)],
                                           key[j], __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        wave_sync();
        const float inv_bw = 1.0f / (float)cv.bw;
        for (uint32_t i = lane; i < area; i += 64) {
            const uint64_t v = w_tile[i];
            if (v != ~0ull) {
                uint32_t r, col;
                tile_rc(i, cv.bw, inv_bw, r, col);
                gu64 *dst = global_ptr(fb) +
                            ((int64_t)(cv.y0 + (int32_t)r) * P.width + cv.x0 + col);
                const uint64_t cur = read_nearest(dst, true);
                if (v < cur)
                    __hip_atomic_fetch_min(dst, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        wave_sync();
        return;
    }
#pragma unroll
    for (int j = 0; j < kGenPpt; ++j) {
        if (!live[j])
            continue;
        int32_t x0, x1, y0, y1;
        cover(px[j], k, P.width, x0, x1);
        cover(py[j], k, P.height, y0, y1);
        for (int32_t yy = y0; yy < y1; ++yy) {
            for (int32_t xx = x0; xx < x1; ++xx) {
                gu64 *dst = global_ptr(fb) + ((int64_t)yy * P.width + xx);
                const uint64_t cur = read_nearest(dst, l2);
                if (key[j] < cur)
                    __hip_atomic_fetch_min(dst, key[j], __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
}

// Splat pass of a wave whose points are all on screen and in range, for maps and
// windows with a threshold per pixel (window_threshold).  False, with acc
// untouched, when that does not hold or the rectangles do not fit `words` words:
//   sums at centres (area) | sums at pixels (covered) | thresholds (covered) |
//   least and greatest threshold over each centre's square (2 area),
// the thresholds giving way to the rows' sums (covered width x rows) in the end.
__device__ __forceinline__ bool hq_points_fast(const Proj &P, const Trans &T, int32_t k,
                                               const Eps &eps, const gu64 *gfb, gu64 *gacc,
                                               const float (&x)[kGenPpt], const float (&y)[kGenPpt],
                                               const float (&z)[kGenPpt],
                                               const uint32_t (&c)[kGenPpt], uint32_t base,
                                               uint32_t words, bool &off)
{
    float fx[kGenPpt], fy[kGenPpt];
    Box box;
    const Where where = window_all<kGenPpt>(P, T, x, y, z, fx, fy, box);
    off = where == kOffScreen;
    if (where != kOnScreen)
        return false;
    const uint32_t lane = threadIdx.x & 63u;
    const WaveTile t = wave_tile(P, box);
    const Covered v = covered_rect(P, box, k);
    if (t.area > words || v.area > words || 3 * t.area + 2 * v.area >= words)   // one word to align
        return false;
    const uint32_t bh = t.area / t.bw;
    const int32_t r = (k - 1) / 2;
    const int32_t ox = (int32_t)v.x0 - (int32_t)t.x0, oy = (int32_t)v.y0 - (int32_t)t.y0;
    const uint32_t cen = base, pix = cen + 8 * t.area, thr = pix + 8 * v.area;
    // 16-byte entries
    const uint32_t ends = (thr + 8 * v.area + 15u) & ~15u;
    typedef __attribute__((address_space(3))) double lf64;
    auto dbl = [](uint32_t a) { return (lf64 *)(uintptr_t)a; };
    auto pixel_of = [&](uint32_t i) {
        uint32_t row, col;
        tile_rc(i, v.w, v.inv_w, row, col);
        return __umul24(v.y0 + row, t.width) + v.x0 + col;
    };
    // the nearest depths of the covered pixels, in flight while the points'
    // depths are computed
    constexpr int kPre = 2;
    uint64_t near[kPre];
#pragma unroll
    for (int n = 0; n < kPre; ++n)
        near[n] = lane + 64 * n < v.area ? gfb[pixel_of(lane + 64 * n)] : 0ull;
    for (uint32_t i = lane; i < t.area + v.area; i += 64)
        *lds_ptr(cen + 8 * i) = 0ull;
    bool in = true;
    double q[kGenPpt];
#pragma unroll
    for (int j = 0; j < kGenPpt; ++j) {
        const double d = depth_of(P, T.td, x[j], y[j], z[j]);
        in = in & (d >= P.dlo[0]) & (d < P.dhi[0]);
        q[j] = floor((d - P.o) * P.s);
    }
    if (wave_any(!in))
        return false;
#pragma unroll
    for (int n = 0; n < kPre; ++n)
        if (lane + 64 * n < v.area)
            *dbl(thr + 8 * (lane + 64 * n)) = window_threshold(P, eps, near[n]);
    for (uint32_t i = lane + 64 * kPre; i < v.area; i += 64)
        *dbl(thr + 8 * i) = window_threshold(P, eps, gfb[pixel_of(i)]);
    wave_sync();
    // the least and the greatest threshold of each centre's square (position of
    // the square's first pixel: centre - r, kept inside the covered rectangle)
    for (uint32_t i = lane; i < t.area; i += 64) {
        uint32_t row, col;
        tile_rc(i, t.bw, t.inv_bw, row, col);
        double lo = __builtin_inf(), hi = -1.0;
        with_size(k, [&](auto kk) {
            for (int dy = 0; dy < kk; ++dy) {
                const int32_t yy = min(max((int32_t)row - oy - r + dy, 0), (int32_t)v.h - 1);
                for (int dx = 0; dx < kk; ++dx) {
                    const int32_t xx = min(max((int32_t)col - ox - r + dx, 0), (int32_t)v.w - 1);
                    const double e = *dbl(thr + 8 * ((uint32_t)yy * v.w + (uint32_t)xx));
                    lo = e < lo ? e : lo;
                    hi = e > hi ? e : hi;
                }
            }
        });
        *dbl(ends + 16 * i) = lo;
        *dbl(ends + 16 * i + 8) = hi;
    }
    wave_sync();
    uint64_t one[kGenPpt];
    bool mixed[kGenPpt];
    bool any_mixed = false;
#pragma unroll
    for (int j = 0; j < kGenPpt; ++j) {
        const uint32_t e = __umul24((uint32_t)(int32_t)fy[j] - t.y0, t.bw) +
                           (uint32_t)(int32_t)fx[j] - t.x0;
        const double lo = *dbl(ends + 16 * e), hi = *dbl(ends + 16 * e + 8);
        one[j] = ((uint64_t)__builtin_amdgcn_perm(1u, c[j], 0x0c040c02u) << 32) |
                 __builtin_amdgcn_perm(1u, c[j], 0x0c010c00u);
        const bool all = q[j] <= lo;
        mixed[j] = !all & (q[j] <= hi);
        any_mixed = any_mixed | mixed[j];
        if (all)
            __hip_atomic_fetch_add(lds_ptr(cen + 8 * e), one[j], __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    if (wave_any(any_mixed)) {
#pragma unroll
        for (int j = 0; j < kGenPpt; ++j) {
            if (!mixed[j])
                continue;
            int32_t x0, x1, y0, y1;
            cover((uint32_t)(int32_t)fx[j], k, P.width, x0, x1);
            cover((uint32_t)(int32_t)fy[j], k, P.height, y0, y1);
            for (int32_t yy = y0; yy < y1; ++yy) {
                const uint32_t at = __umul24((uint32_t)yy - v.y0, v.w) - v.x0;
                for (int32_t xx = x0; xx < x1; ++xx) {
                    const uint32_t e = at + (uint32_t)xx;
                    if (q[j] <= *dbl(thr + 8 * e))
                        __hip_atomic_fetch_add(lds_ptr(pix + 8 * e), one[j], __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
        }
    }
    wave_sync();
    // sums over the centres of each row that cover a column, then over the rows
    // that cover a pixel: centres outside the tile do not count
    const uint32_t line = thr;
    with_size(k, [&](auto kk) {
        for (uint32_t i = lane; i < v.w * bh; i += 64) {
            uint32_t row, col;
            tile_rc(i, v.w, v.inv_w, row, col);
            uint64_t sum = 0;
            for (int d = 0; d < kk; ++d) {
                const uint32_t cc = (uint32_t)((int32_t)col + ox + r - d);   // < 0: large
                const uint64_t e = *lds_ptr(cen + 8 * (row * t.bw + (cc < t.bw ? cc : 0u)));
                sum += cc < t.bw ? e : 0ull;
            }
            *lds_ptr(line + 8 * i) = sum;
        }
    });
    wave_sync();
    for (uint32_t i = lane; i < v.area; i += 64) {
        uint32_t row, col;
        tile_rc(i, v.w, v.inv_w, row, col);
        uint64_t sum = *lds_ptr(pix + 8 * i);
        with_size(k, [&](auto kk) {
            for (int d = 0; d < kk; ++d) {
                const uint32_t rr = (uint32_t)((int32_t)row + oy + r - d);
                const uint64_t e = *lds_ptr(line + 8 * ((rr < bh ? rr : 0u) * v.w + col));
                sum += rr < bh ? e : 0ull;
            }
        });
        if (sum != 0ull) {   // unpack into the accumulator's two words
            gu64 *dst = gacc + 2 * (uint64_t)(__umul24(v.y0 + row, t.width) + v.x0 + col);
            const uint64_t a0 = (sum & 0xFFFFull) | (((sum >> 16) & 0xFFFFull) << 32);
            const uint64_t a1 = ((sum >> 32) & 0xFFFFull) | ((sum >> 48) << 32);
            __hip_atomic_fetch_add(dst, a0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_fetch_add(dst + 1, a1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    return true;
}

template <bool PW>
__global__ void __launch_bounds__(kGenBlock) k_hq_points(Pts p, Proj P, int32_t k, Eps eps,
                                                         const uint64_t *__restrict__ fb,
                                                         uint64_t *__restrict__ acc,
                                                         uint32_t words)
{
    extern __shared__ uint64_t s_waves[];
    uint64_t *w_tile = s_waves + (threadIdx.x >> 6) * words;   // packed sums
    uint64_t *w_qmin = w_tile + words / 2;                     // nearest depths
    const int64_t base = (int64_t)blockIdx.x * kGenBlock * kGenPpt;
    float x[kGenPpt], y[kGenPpt], z[kGenPpt];
    uint32_t c[kGenPpt];
    load_points_nan<kGenPpt>(p, base, x, y, z, c);
    if (!PW && window_exact(P, eps)) {
        bool off;
        if (hq_points_fast(P, lane_trans(P), k, eps, (const gu64 *)global_ptr(fb), global_ptr(acc),
                           x, y, z, c, lds_addr(w_tile), words, off) ||
            off)
            return;
    }
    const uint32_t eps_num = eps.num, eps_den = eps.den;
    uint32_t px[kGenPpt], py[kGenPpt];
    uint64_t q[kGenPpt];
    bool live[kGenPpt];
#pragma unroll
    for (int j = 0; j < kGenPpt; ++j) {
        uint32_t a = 0, b = 0;
        uint64_t qq = 0;
        live[j] = fragment<PW>(P, x[j], y[j], z[j], a, b, qq);
        px[j] = a;
        py[j] = b;
        q[j] = qq;
    }
    const Cover cv = wave_cover(wave_box<kGenPpt>(px, py, live), k, P.width, P.height,
                                words / 2);
    const uint32_t lane = threadIdx.x & 63u;
    if (cv.tiled) {
        // the nearest depth of every pixel of the rectangle, read once with
        // coalesced row loads, then looked up in LDS per covered pixel
        const uint32_t area = cv.bw * cv.bh;
        const float inv_bw = 1.0f / (float)cv.bw;
        for (uint32_t i = lane; i < area; i += 64) {
            uint32_t r, col;
            tile_rc(i, cv.bw, inv_bw, r, col);
            w_qmin[i] = fb[__umul24((uint32_t)cv.y0 + r, (uint32_t)P.width) + cv.x0 + col] >> 24;
            w_tile[i] = 0ull;
        }
        wave_sync();
#pragma unroll
        for (int j = 0; j < kGenPpt; ++j) {
            if (!live[j])
                continue;
            const uint32_t col = c[j];
            const uint64_t w = (uint64_t)(col & 0xFFu) | ((uint64_t)((col >> 8) & 0xFFu) << 16) |
                               ((uint64_t)((col >> 16) & 0xFFu) << 32) | (1ull << 48);
            int32_t x0, x1, y0, y1;
            cover(px[j], k, P.width, x0, x1);
            cover(py[j], k, P.height, y0, y1);
            for (int32_t yy = y0; yy < y1; ++yy) {
                const uint32_t row = __umul24((uint32_t)(yy - cv.y0), cv.bw) - (uint32_t)cv.x0;
                for (int32_t xx = x0; xx < x1; ++xx) {
                    const uint32_t t = row + (uint32_t)xx;
                    if (!in_window_live<PW>(P, eps_num, eps_den, q[j], w_qmin[t], true))
                        continue;
                    __hip_atomic_fetch_add(&w_tile[t], w, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
        }
        wave_sync();
        for (uint32_t i = lane; i < area; i += 64) {
            const uint64_t sw = w_tile[i];
            if (sw != 0ull) {   // unpack into the accumulator's two words
                const uint64_t a0 = (sw & 0xFFFFull) | (((sw >> 16) & 0xFFFFull) << 32);
                const uint64_t a1 = ((sw >> 32) & 0xFFFFull) | ((sw >> 48) << 32);
                uint32_t r, col;
                tile_rc(i, cv.bw, inv_bw, r, col);
                uint64_t *dst =
                    acc + 2 * (uint64_t)(__umul24((uint32_t)cv.y0 + r, (uint32_t)P.width) +
                                         cv.x0 + col);
                __hip_atomic_fetch_add(dst, a0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_fetch_add(dst + 1, a1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        wave_sync();
        return;
    }
    // the squares spread too far for the tile: global reads and atomics
#pragma unroll
    for (int j = 0; j < kGenPpt; ++j) {
        if (!live[j])
            continue;
        const uint32_t col = c[j];
        const uint64_t w0 = (uint64_t)(col & 0xFFu) | ((uint64_t)((col >> 8) & 0xFFu) << 32);
        const uint64_t w1 = (uint64_t)((col >> 16) & 0xFFu) | (1ull << 32);
        int32_t x0, x1, y0, y1;
        cover(px[j], k, P.width, x0, x1);
        cover(py[j], k, P.height, y0, y1);
        for (int32_t yy = y0; yy < y1; ++yy) {
            for (int32_t xx = x0; xx < x1; ++xx) {
                const uint64_t pp = __umul24((uint32_t)yy, (uint32_t)P.width) + (uint32_t)xx;
                if (!in_window<PW>(P, eps_num, eps_den, q[j], fb[pp] >> 24))
                    continue;
                __hip_atomic_fetch_add(acc + 2 * pp, w0, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_fetch_add(acc + 2 * pp + 1, w1, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
}

}  // namespace

hipError_t launch_raster_points(const Pts &p, const Proj &P, int32_t k, uint64_t *fb,
                                hipStream_t s)
{
    Range r("rz depth pass (k x k points)");
    if (p.n == 0)
        return hipSuccess;
    const dim3 grid((uint32_t)((p.n + kGenBlock * kGenPpt - 1) / (kGenBlock * kGenPpt)));
    const size_t lds = (kGenBlock / 64) * kWaveTileWords * sizeof(uint64_t);
    if (P.zkind == RZ_DEPTH_GL24)
        hipLaunchKernelGGL((k_raster_points<false, RZ_DEPTH_GL24>), grid, dim3(kGenBlock), lds, s,
                           p, P, k, fb);
    else if (P.zkind == RZ_DEPTH_F32REV)
        hipLaunchKernelGGL((k_raster_points<false, RZ_DEPTH_F32REV>), grid, dim3(kGenBlock), lds,
                           s, p, P, k, fb);
    else if (P.nr != 0)
        hipLaunchKernelGGL((k_raster_points<true, 0>), grid, dim3(kGenBlock), lds, s, p, P, k, fb);
    else
        hipLaunchKernelGGL((k_raster_points<false, 0>), grid, dim3(kGenBlock), lds, s, p, P, k,
                           fb);
    return hipGetLastError();
}

hipError_t launch_hq_points(const Pts &p, const Proj &P, int32_t k, uint32_t eps_num,
                            uint32_t eps_den, const uint64_t *fb, uint64_t *acc, hipStream_t s)
{
    Range r("rz splat accumulate pass (k x k points)");
    if (p.n == 0)
        return hipSuccess;
    const dim3 grid((uint32_t)((p.n + kGenBlock * kGenPpt - 1) / (kGenBlock * kGenPpt)));
    const Eps eps{eps_num, eps_den, 1.0 / (double)eps_den};
    const uint32_t words = k <= 5 ? kWaveTileWords : kHqWordsLarge;
    const size_t lds = (kGenBlock / 64) * words * sizeof(uint64_t);
    if (P.nr != 0)
        hipLaunchKernelGGL((k_hq_points<true>), grid, dim3(kGenBlock), lds, s, p, P, k, eps, fb,
                           acc, words);
    else
        hipLaunchKernelGGL((k_hq_points<false>), grid, dim3(kGenBlock), lds, s, p, P, k, eps, fb,
                           acc, words);
    return hipGetLastError();
}

}  // namespace rz
