// Internal declarations shared by the host side of the library and the
// kernel launchers.  Not part of the public C ABI (that is include/rz.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rz {

// Per-view constants of one rasterization, derived on the host in double
// precision and passed to the kernels by value.
struct Proj {
    float m[12];          // rows 0, 1 and 3 of (float)VP, row-major
    float fw, fh;         // framebuffer size as float
    float hw, hh;         // half of it
    float mz[4];          // row 2 of (float)VP (window depth encodings)
    float nearf;          // near as float (reversed float depth)
    int32_t zkind;        // 0: integer map (linear, scale, piecewise);
                          // RZ_DEPTH_GL24 or RZ_DEPTH_F32REV otherwise
    double v[4];          // row 3 of VP in double: the depth row
    double near_, far_;
    double o, s;          // q = floor((d - o) * s)
    uint64_t z0;          // floor(o * s)
    int32_t width, height;
    // piecewise depth map: nr > 0 selects it
    int32_t nr;
    int32_t pad_;
    double rb[8];         // range starts
    double rs[8];         // values per unit
    double rinv[8];       // 1 / rs
    uint64_t rbase[9];    // first integer of each range; rbase[nr] = 2^40 - 1
    // Range k of the depth map (0 for the linear and scale maps): a depth in
    // [dlo[k], dhi[k]) is in [near, far), lies in the range and has a q of at
    // most 2^40 - 2 without the clamp.
    double dlo[8], dhi[8];
    double z0d;           // z0 as a double (exact when wfp is set)
    int32_t wfp;          // z0 < 2^52: the eps window may be pre-tested in double
    int32_t pad2_;
};

// Launch shape of the point kernels.  The defaults are those of the depth
// pass; the splat accumulate pass defaults to kHqTune (measured on the
// 50M-point terrain: 64 threads, 8 points each, the small per-wave tile).
struct Tune {
    int block = 64;        // threads per workgroup: 64, 128, 256 or 512
    int ppt = 16;          // points per thread: 4, 8 or 16
    int early_out = 1;     // read the framebuffer before the atomic
    int xcd_remap = 0;     // give each XCD a contiguous range of chunks
    int bin = 2;           // 0 none, 1 workgroup LDS tile, 2 per-wave LDS tile,
                           // 3 the small per-wave tile
    int by_size = 1;       // library default: small clouds take kSmallTune
    int read_first = 1;    // per-wave tiles: early-out reads also beside the tile
};

constexpr Tune kHqTune = {64, 8, 1, 0, 3, 1};
// Clouds of fewer points than this: four times the waves, each done sooner.  At
// the default shapes they are one or two rounds of 4096 waves of 1024 points (5120
// of 512 in the splat pass), so that a pass lasts as long as its slowest waves.
// Frames of the terrain at 1920x1080, default shape / this one: 0.5M points 25.1 /
// 21.5 us (splat 64.9 / 56.3), 2M 29.7 / 27.1 (73.3 / 66.4), 5M 36.1 / 31.5 (81.9 /
// 77.3), 10M 47.4 / 44.6 (101.7 / 100.6), 20M 71.9 / 72.4 (149.0 / 152.9).  In the
// depth pass the four waves of a workgroup share a tile where they cover the same
// pixels (raster_chunk_group).
constexpr int64_t kSmallCloud = 8 << 20;
constexpr Tune kSmallTune = {256, 4, 1, 0, 3, 1};
// Screens of at most this many pixels, of which a wave of either shape has a fragment
// for nearly every one: the splat pass's time is the number of waves, whose sums of one
// pixel follow each other, and it keeps the larger ones.  Frames of spheres in random
// order, 256 / 512 points a wave: 8 x 8 pixels 0.3M points 41.2 / 35.5 us, 0.9M 105 / 84.8,
// 3M 328 / 242; 16 x 16 40.1 / 36.0, 96.5 / 86.4, 299 / 243.
constexpr int64_t kFewPixels = 512;
// Clouds of fewer points than this do not fill the device, and a fragment beside
// a tile (a cloud in no spatial order) costs the latencies of its early-out read and
// of its atomic in turn: they go without the read, which would seldom save the atomic,
// since all waves start at once.  Frames, with the read / without: spheres at 1024x768
// 0.2M points 19.3 / 17.0 us, 0.4M 29.5 / 26.6, 0.8M 50.9 / 42.0, 1M 59.5 / 56.9, 1.3M
// 69.7 / 72.4, 2M 87.7 / 108.7; shuffled terrain at 2560x1440 0.4M 37.0 / 31.7, 1M 62.8 /
// 56.7, 2M 98.1 / 95.5, at 320x200 0.4M 48.0 / 34.3, 1M 106.5 / 78.1, 1.6M 123 / 123, 2M
// 131 / 151; spheres of 0.7M on 256 x 256 pixels 90.5 / 40.7, 160 x 160 140 / 61, 96 x 96
// 219 / 75, 64 x 64 255 / 98 (on fewer pixels the waves share a tile).
constexpr int64_t kUnreadCloud = 1 << 20;
constexpr Tune kUnreadTune = {256, 4, 1, 0, 3, 1, 0};

// The splat window's eps = num / den, with 1 / den rounded once.
struct Eps {
    uint32_t num, den;
    double inv_den;
};

// Whether a rectangle of `area` pixels fits a tile of `words` 8-byte words at
// 1 << sh bytes per pixel (sh >= 3).  A rectangle of a 32768 x 32768 screen has up
// to 2^30 pixels: 32 bits hold its area, but not its bytes.
__host__ __device__ constexpr bool tile_fits(uint32_t area, uint32_t words, uint32_t sh)
{
    return area <= words >> (sh - 3);
}

constexpr uint64_t kDepthOnes = 0xFFFFFFFFFF000000ull;
constexpr uint64_t kRgbMask = 0xFFFFFFull;
constexpr uint64_t kHqCountMax = 16843009ull;   // floor((2^32 - 1) / 255)

// Point planes on the device.
struct Pts {
    const float *x, *y, *z;
    const uint32_t *rgb;
    int64_t n;
};

hipError_t launch_raster_min(const Pts &p, const Proj &P, uint64_t *fb, const Tune &t,
                             hipStream_t s);
hipError_t launch_hq_accum(const Pts &p, const Proj &P, uint32_t eps_num, uint32_t eps_den,
                           const uint64_t *fb, uint64_t *acc, const Tune &t, hipStream_t s);
hipError_t launch_resolve_min(uint64_t *fb, int64_t npix, uint32_t bg, uint32_t *img,
                              hipStream_t s);
hipError_t launch_resolve_hq(uint64_t *fb, uint64_t *acc, int64_t npix, uint32_t bg,
                             uint32_t *img, uint32_t *status, hipStream_t s);
hipError_t launch_clear(uint64_t *fb, uint64_t *acc, int64_t npix, uint32_t bg, hipStream_t s);
// Points of size k >= 1 and every depth encoding (one fragment per covered
// pixel, early-out plus global atomics).
hipError_t launch_raster_points(const Pts &p, const Proj &P, int32_t k, uint64_t *fb,
                                hipStream_t s);

// One view of a multi-view pass (an entry of a device table): the batch
// engine's groups and the server's merged requests.
struct MvView {
    Proj P;
    uint64_t *fb;
    uint64_t *acc;
    Eps eps;
};
constexpr int kMaxGroupViews = 8;   // views per multi-view launch

// Depth passes (hq false) or accumulate passes (hq true) of views[0 .. nv)
// (a device table, nv <= kMaxGroupViews) over the points, each chunk of
// points loaded once for all of them.  pw: some view uses a piecewise map.
hipError_t launch_multiview(bool hq, bool pw, const Pts &p, const MvView *views, int32_t nv,
                            const Tune &t, hipStream_t s);
hipError_t launch_hq_points(const Pts &p, const Proj &P, int32_t k, uint32_t eps_num,
                            uint32_t eps_den, const uint64_t *fb, uint64_t *acc, hipStream_t s);

}  // namespace rz
