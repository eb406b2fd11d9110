"""Waves that leave the kernels' common path, against the oracle: rectangles of large
screens, sums at the limit of the tile's words, windows and depth ranges that
split a wave at every launch shape."""
import sys

import numpy as np
import pytest

from paper_1908_02681_amd import gen
from tests.test_gpu_paths import rectangle_scene

pytestmark = pytest.mark.gpu


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def rz():
    from paper_1908_02681_amd import rz as m
    m.load()
    return m


@pytest.mark.parametrize("size,shape", [((32768, 16384), None), ((16384, 16384), (64, 16, 1, 0, 2)),
                                        ((16384, 16384), (64, 16, 1, 0, 3))])
def test_splat_waves_across_large_screens(rz, oracle, size, shape):
    """Every wave spans a screen whose pixels, at the tile's 8 or 16 bytes each, take
    exactly 2^32 bytes: the sums of every touched pixel, from the oracle's fragments,
    and no count anywhere else."""
    import torch
    W, H = size
    n = 20_011
    say(f"[large screen] {size} {shape}")
    c, v = rectangle_scene(W, H, n, 3, W=W, H=H, ox=0, oy=0)
    half = np.arange(n // 2) * 2   # half of the points again where a neighbour lies, a little deeper
    half = half[(half % 64 != 2) & (half % 64 != 40)]
    for a in (c.x, c.y, c.z):
        a[half + 1] = a[half] * np.float32(1.005)
    pix, q = oracle.fragments(c.x, c.y, c.z, v.vp, v.near, v.far, W, H)
    live = pix >= 0
    assert live.mean() > 0.95
    o, s, z0 = oracle.depth_constants(v.vp, v.near, v.far, W, H)[:3]
    p, d, col = pix[live], q[live].astype(object), c.rgb[live]
    near = {}
    for i, k in zip(p, d):
        near[i] = min(near.get(i, k), k)
    want = {}
    for i, k, w in zip(p, d, col):
        if 100 * (k - near[i]) <= near[i] + int(z0):
            t = want.setdefault(i, [0, 0, 0, 0])
            for ch in range(3):
                t[ch] += (int(w) >> (8 * ch)) & 0xFF
            t[3] += 1
    assert max(t[3] for t in want.values()) > 1
    pts = rz.Points.from_cloud(c)
    rz.reset_launch() if shape is None else rz.set_launch(*shape)
    try:
        fb, acc, _, _ = rz.rasterize_hq_splat(pts, v, keep_keys=True)
    finally:
        rz.reset_launch()
    idx = np.array(sorted(want), np.int64)
    pairs = acc.view(-1, 2)
    got = rz.unpack_acc(pairs[torch.from_numpy(idx).cuda()].reshape(-1))
    written = int((pairs[:, 1] != 0).sum().item())
    del fb, acc, pairs
    torch.cuda.empty_cache()
    assert np.array_equal(got, np.array([want[i] for i in idx], got.dtype))
    assert written == len(idx)


@pytest.mark.parametrize("kind", [3, 4])
@pytest.mark.parametrize("k", [1, 3])
def test_float_encodings_with_far_at_infinity(rz, oracle, kind, k):
    """A far plane beyond any depth that a 40-bit map could hold: keys of the float
    encodings, ordered and in no order."""
    c = gen.terrain(60_000, 52, extent=100.0, amplitude=10.0, wavelength=40.0)
    t = gen.orbit_views(1, 13, [(160, 120)], extent=100.0, rmin=60.0, rmax=120.0, near=0.5,
                        far=400.0)[0]
    v = gen.View(t.vp, t.near, 1e30, t.width, t.height)
    for cloud in (c, gen.shuffle(c, 3)):
        want, _ = oracle.render_atomicmin(cloud.x, cloud.y, cloud.z, cloud.rgb, v.vp, v.near, v.far,
                                          v.width, v.height, kind, point_size=k)
        assert (want != np.uint64(oracle.clear_value(0))).mean() > 0.1
        fb, _, _, _ = rz.rasterize_points(rz.Points.from_cloud(cloud), v, (kind, 0.0), point_size=k,
                                          keep_keys=True)
        assert np.array_equal(rz.to_u64(fb), want)


def render_all(rz, oracle, c, v, depth=(0, 0.0), eps=(1, 100), shape=None, sizes=(1, 2, 3)):
    """Keys, splat sums and batch images of one scene against the oracle's."""
    args = (c.x, c.y, c.z, c.rgb, v.vp, v.near, v.far, v.width, v.height, *depth)
    pts = rz.Points.from_cloud(c)
    rz.reset_launch() if shape is None else rz.set_launch(*shape)
    try:
        for k in sizes:
            keys, img = oracle.render_atomicmin(*args, point_size=k)
            fb, _, _, _ = rz.rasterize_points(pts, v, depth, point_size=k, keep_keys=True)
            assert np.array_equal(rz.to_u64(fb), keys), (k, "keys")
            _, sums, himg = oracle.render_hq(*args, eps=eps, point_size=k)
            _, acc, _, _ = rz.rasterize_points(pts, v, depth, True, eps, k, keep_keys=True)
            assert np.array_equal(rz.unpack_acc(acc), sums), (k, "sums")
            if k == 1:
                b = rz.Batch(pts, [v, v, v], [0, 1, 0], depth=depth, eps=eps, launch=shape)
                b.run()
                got = b.images()
                assert np.array_equal(got[0], img) and np.array_equal(got[2], img)
                assert np.array_equal(got[1], himg)
    finally:
        rz.reset_launch()


SHAPES = [None, (64, 8, 1, 0, 3), (64, 16, 1, 0, 2)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("what", ["behind", "at zero", "a few in front", "a few at zero", "nan"])
def test_waves_behind_the_camera(rz, oracle, what, shape):
    """Whole waves with w < 0, w = -0 and w NaN beside waves in front, and waves of which a
    few points are in front of the camera or in its plane (w = 0)."""
    n = 6000
    c, v = rectangle_scene(40, 30, n, 8)
    part = np.arange(n // 4, 3 * n // 4)
    if what == "nan":
        c.z[part] = np.nan
    else:
        c.x[part], c.y[part], c.z[part] = -c.x[part], -c.y[part], -c.z[part]
    if what == "at zero":
        c.x[part], c.y[part], c.z[part] = -np.abs(c.x[part]), -np.abs(c.y[part]), -0.0
        v.vp[3, 3] = -0.0   # w = -0 for them
    if what == "a few in front":
        some = part[::57]
        c.x[some], c.y[some], c.z[some] = -c.x[some], -c.y[some], -c.z[some]
    if what == "a few at zero":
        c.z[part[::57]] = 0.0
    render_all(rz, oracle, c, v, shape=shape)


PIECES = [(0, 0.0), (2, ((0.0, 1e9), (2.015, 1e6), (10.0, 1e3))), (3, 0.0), (4, 0.0)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("depth", PIECES)
@pytest.mark.parametrize("wh", [(9, 7), (41, 25), (300, 200)])
def test_waves_across_depth_ranges(rz, oracle, wh, depth, shape):
    """Waves of which some points lie before near, beyond far or in another range of the
    depth map, over rectangles inside the tile (four copies and one) and beside it,
    partly off screen too."""
    for i, (ox, oy) in enumerate([(37, 21), (-3, -2)]):
        c, v = rectangle_scene(*wh, n=3001, seed=20 + i, ox=ox, oy=oy, outside=300)
        v.near, v.far = 2.005, 2.05   # z is 2 to 2.03 or about 2.5
        args = (c.x, c.y, c.z, c.rgb, v.vp, v.near, v.far, v.width, v.height, *depth)
        pts = rz.Points.from_cloud(c)
        keys, img = oracle.render_atomicmin(*args)
        rz.reset_launch() if shape is None else rz.set_launch(*shape)
        try:
            fb, _ = rz.rasterize_atomicmin(pts, v, depth, keep_keys=True)
        finally:
            rz.reset_launch()
        assert np.array_equal(rz.to_u64(fb), keys), (ox, oy)
        if depth[0] < 3:
            b = rz.Batch(pts, [v, v], [0, 0], depth=depth, launch=shape)
            b.run()
            assert all(np.array_equal(g, img) for g in b.images())


@pytest.mark.parametrize("shape", SHAPES)
def test_waves_of_extreme_w(rz, oracle, shape):
    """Points whose w is denormal or at least 2^126, where the reciprocal takes the IEEE
    quotient, among ordinary ones and alone."""
    n = 4000
    c, v = rectangle_scene(30, 20, n, 12)
    v.near, v.far = 1e-41, 1e39
    scale = np.ones(n)
    scale[100:1100:7] = 1e38 / 2
    scale[1500:2200] = 1e38 / 2
    scale[2300:3000:5] = 3e-39
    scale[3200:3900] = 3e-39
    for a in (c.x, c.y, c.z):
        a[:] = (a.astype(np.float64) * scale).astype(np.float32)
    pix, _ = oracle.fragments(c.x, c.y, c.z, v.vp, v.near, v.far, v.width, v.height)
    assert (pix[1500:2200] >= 0).any() and (pix[3200:3900] >= 0).any()
    render_all(rz, oracle, c, v, shape=shape)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("depth", PIECES[:2])
def test_runs_of_one_pixel_beside_the_tile(rz, oracle, depth, shape):
    """Runs of 1 to 6 consecutive points in one pixel, some of them out of range, in waves
    spread too far for any tile."""
    n = 5003
    c, v = rectangle_scene(350, 250, n, 33)
    v.far = 2.4
    rng = np.random.default_rng(34)
    src = np.repeat(np.arange(n), rng.integers(1, 7, n))[:n]
    deeper = rng.choice([1.0, 1.001, 1.003, 1.3], n, p=[0.3, 0.3, 0.3, 0.1]).astype(np.float32)
    for a in (c.x, c.y, c.z):
        a[:] = a[src] * deeper   # along the ray: the same pixel, or beyond far
    render_all(rz, oracle, c, v, depth=depth, shape=shape, sizes=(1, 2))


@pytest.mark.parametrize("depth", PIECES)
@pytest.mark.parametrize("wh", [(1, 1), (16, 16), (17, 16), (32, 32), (33, 32), (60, 40)])
def test_waves_that_share_a_tile(rz, oracle, wh, depth):
    """Small clouds whose workgroups have waves over the same pixels (one tile for all, with
    four copies and one), beside others: waves off screen, behind the camera, of extreme
    w and elsewhere on the screen, in every place of the workgroup; into a framebuffer that
    holds keys already."""
    n = 16 * 256 + 77
    c, v = rectangle_scene(*wh, n, 41, outside=200)
    v.near, v.far = 2.005, 1e39
    if depth[0] == 0:
        v.far = 2.6
    rng = np.random.default_rng(42)
    for i, what in enumerate(["", "off", "", "behind", "behind", "off", "off", "", "far", "", "",
                              "far", "huge", "", "off", ""]):
        w = slice(256 * i, 256 * (i + 1))
        if what == "off":
            c.x[w] += 4 * np.abs(c.z[w])
        elif what == "behind":
            for a in (c.x, c.y, c.z):
                a[w] = -a[w]
        elif what == "far":
            c.x[w] += (0.5 * c.z[w]).astype(np.float32)
        elif what == "huge" and depth[0] != 0:
            for a in (c.x, c.y, c.z):
                a[256 * i + 5:256 * (i + 1):9] *= np.float32(5e37)
    v2 = gen.View(v.vp, v.near, v.far, v.width, v.height)
    if depth[0] == 2:
        v2.far = 2.6
    pts = rz.Points.from_cloud(c)
    keys, _ = oracle.render_atomicmin(c.x, c.y, c.z, c.rgb, v2.vp, v2.near, v2.far, v2.width,
                                      v2.height, *depth)
    fb, _ = rz.new_framebuffer(v2, 0)
    for _ in range(2):
        rz.rasterize_atomicmin(pts, v2, depth, fb=fb, keep_keys=True)
        assert np.array_equal(rz.to_u64(fb), keys)
    some = rng.permutation(n)[:1500]   # fewer, in another order, into the same keys
    c2 = gen.Cloud(c.x[some], c.y[some], c.z[some], c.rgb[some] ^ np.uint32(0x010101))
    want = oracle.render_atomicmin(np.r_[c.x, c2.x], np.r_[c.y, c2.y], np.r_[c.z, c2.z],
                                   np.r_[c.rgb, c2.rgb], v2.vp, v2.near, v2.far, v2.width,
                                   v2.height, *depth)[0]
    rz.rasterize_atomicmin(rz.Points.from_cloud(c2), v2, depth, fb=fb, keep_keys=True)
    assert np.array_equal(rz.to_u64(fb), want)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("depth,eps", [((0, 0.0), (1, 100)), ((0, 0.0), (1, 4097)),
                                       ((2, ((0.0, 1e9), (2.015, 1e6), (10.0, 1e3))), (1, 100))])
@pytest.mark.parametrize("wh", [(9, 7), (24, 20), (41, 25), (300, 200)])
def test_splats_across_depth_ranges(rz, oracle, wh, depth, eps, shape):
    """Sums of waves of which some points lie before near, beyond far or in another range,
    under windows with a threshold per pixel and without, inside the tile and beside it,
    partly off screen too."""
    for i, (ox, oy) in enumerate([(37, 21), (-3, -2)]):
        c, v = rectangle_scene(*wh, n=3001, seed=50 + i, ox=ox, oy=oy, outside=300, behind=40)
        v.near, v.far = 2.005, 2.05
        keys, sums, himg = oracle.render_hq(c.x, c.y, c.z, c.rgb, v.vp, v.near, v.far, v.width,
                                            v.height, *depth, eps=eps)
        pts = rz.Points.from_cloud(c)
        rz.reset_launch() if shape is None else rz.set_launch(*shape)
        try:
            fb, acc, _, _ = rz.rasterize_hq_splat(pts, v, depth, eps, keep_keys=True)
        finally:
            rz.reset_launch()
        assert np.array_equal(rz.to_u64(fb), keys), (ox, oy)
        assert np.array_equal(rz.unpack_acc(acc), sums), (ox, oy)
        b = rz.Batch(pts, [v, v], [1, 1], depth=depth, eps=eps, launch=shape)
        b.run()
        assert all(np.array_equal(g, himg) for g in b.images())


@pytest.mark.parametrize("shape", [None, (64, 8, 1, 0, 3), (128, 8, 1, 0, 2), (64, 16, 1, 0, 2)])
@pytest.mark.parametrize("depth,eps", [((0, 0.0), (1, 100)), ((0, 0.0), (1, 4097)),
                                       ((2, ((0.0, 1e9), (10.0, 1e6))), (1, 100))])
@pytest.mark.parametrize("rgb", [0xFFFFFF, 0xFF00FF, 0x00FF00])
def test_splat_word_limits_under_every_window(rz, rgb, depth, eps, shape):
    """Every point in one pixel with one colour, under windows with a threshold per pixel
    (16-bit fields in copies of the tile) and under windows and maps without (17-bit fields in
    one copy): the sums are n times each channel and n, with no carry from field to field,
    also where a thread's points are summed first."""
    import torch
    view = gen.View(np.diag([1.0, 1.0, 0.0, 0.0]) + np.array(
        [[0, 0, 0, 0], [0, 0, 0, 0], [0, 0, 0, 0], [0, 0, -1.0, 0]]), 1.0, 100.0, 2, 2)
    n = 5 * 64 * 16 * 8 + 77
    pts = rz.Points(torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda"),
                    torch.full((n,), -10.0, device="cuda"),
                    torch.full((n,), rgb, dtype=torch.int32, device="cuda"))
    rz.reset_launch() if shape is None else rz.set_launch(*shape)
    try:
        _, acc, _, _ = rz.rasterize_hq_splat(pts, view, depth, eps, keep_keys=True)
    finally:
        rz.reset_launch()
    sums = rz.unpack_acc(acc)
    hit = np.flatnonzero(sums[:, 3])
    assert hit.size == 1
    want = [n * (rgb & 0xFF), n * ((rgb >> 8) & 0xFF), n * ((rgb >> 16) & 0xFF), n]
    assert sums[hit[0]].tolist() == want


@pytest.mark.parametrize("wh", [(8, 8), (32, 16), (27, 19)])
@pytest.mark.parametrize("n", [1, 513, 5003])
def test_splats_on_few_pixels(rz, oracle, n, wh):
    """Screens on both sides of the size from which small clouds take the small shape."""
    c, v = rectangle_scene(*wh, n, 60, W=wh[0], H=wh[1], ox=0, oy=0)
    render_all(rz, oracle, c, v)
