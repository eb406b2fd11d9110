"""GPU against the oracle at the edges of the kernels' own decisions: plane
alignment, screen edges, tile limits, launch sizes."""
import numpy as np
import pytest

from paper_1908_02681_amd import gen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rz():
    from paper_1908_02681_amd import rz as m
    m.load()
    return m


def full_render(oracle, c, v, bg=0, **kw):
    """Oracle keys, image, splat sums and splat image of one scene."""
    keys, img = oracle.render_atomicmin(c.x, c.y, c.z, c.rgb, v.vp, v.near, v.far, v.width,
                                        v.height, bg=bg, **kw)
    _, sums, himg = oracle.render_hq(c.x, c.y, c.z, c.rgb, v.vp, v.near, v.far, v.width, v.height,
                                     bg=bg, **kw)
    return keys, img, sums, himg


@pytest.mark.parametrize("offs", [(1, 1, 1, 1), (2, 2, 2, 2), (3, 3, 3, 3), (0, 1, 2, 3)])
def test_planes_at_any_dword_offset(rz, oracle, offs):
    """Planes that start 1 to 3 elements past a 16-byte boundary, alike or
    each on its own, through every kernel that loads points."""
    n = 20_003
    c = gen.terrain(n, 11, extent=50.0, amplitude=5.0, wavelength=20.0)
    v = gen.terrain_view(90, 70, extent=50.0, distance=60.0, near=0.5, far=400.0)
    import torch
    planes = []
    for a, o in zip((c.x, c.y, c.z, c.rgb.view(np.int32)), offs):
        t = torch.zeros(n + 4, dtype=torch.float32 if a.dtype == np.float32 else torch.int32,
                        device="cuda")
        t[o:o + n] = torch.from_numpy(np.ascontiguousarray(a)).cuda()
        planes.append(t[o:o + n])
    pts = rz.Points(*planes)
    keys, img, sums, himg = full_render(oracle, c, v)
    fb, _ = rz.rasterize_atomicmin(pts, v, keep_keys=True)
    assert np.array_equal(rz.to_u64(fb), keys)
    for fn in (rz.rasterize_hq_splat, lambda p, w: rz.rasterize_sorted(p, w, hq=True)):
        assert np.array_equal(rz.to_u32(fn(pts, v)[2]), himg)
    b = rz.Batch(pts, [v, v], [rz.RZ_MODE_ATOMICMIN, rz.RZ_MODE_HQ])
    b.run()
    got = b.images()
    assert np.array_equal(got[0], img) and np.array_equal(got[1], himg)
    k2, _ = oracle.render_atomicmin(c.x, c.y, c.z, c.rgb, v.vp, v.near, v.far, v.width, v.height,
                                    point_size=2)
    fb2, _, _, _ = rz.rasterize_points(pts, v, point_size=2, keep_keys=True)
    assert np.array_equal(rz.to_u64(fb2), k2)


def rectangle_scene(w, h, n, seed, W=400, H=300, ox=37, oy=21, outside=0, behind=0,
                    pile=False):
    """n points over a w x h pixel rectangle (its corners in every 64 points),
    most of them white, depths spread over a few eps windows; `outside` points
    beyond far and `behind` points behind the camera in the middle of the cloud;
    pile: all points but the corners in one pixel, within one window."""
    rng = np.random.default_rng(seed)
    px, py = ox + rng.integers(0, w, n), oy + rng.integers(0, h, n)
    if pile:
        px[:], py[:] = ox, oy
    k = np.arange(n) % 64
    px[k == 3], py[k == 3] = ox, oy
    px[k == 40], py[k == 40] = ox + w - 1, oy + h - 1
    z = (rng.choice([2.0, 2.01, 2.02, 2.5], n) * rng.uniform(1.0, 1.004, n)).astype(np.float32)
    if pile:
        z[:] = 2.0
    m = n // 2
    z[m:m + outside] = 60.0
    x = ((2 * (px + 0.5) / W - 1) * z).astype(np.float32)
    y = ((2 * (py + 0.5) / H - 1) * z).astype(np.float32)
    z[m + 100:m + 100 + behind] *= -1
    vp = np.zeros((4, 4))
    vp[0, 0] = vp[1, 1] = vp[3, 2] = 1.0   # clip = (x, y, ., z)
    vp[2, 2] = 1.0
    rgb = np.full(n, 0xFFFFFF, np.uint32)
    if not pile:
        rgb[::5] = rng.integers(0, 1 << 24, rgb[::5].size)
    return gen.Cloud(x, y, z, rgb), gen.View(vp, 0.5, 50.0, W, H)


TILES = [(1, 1), (2, 1), (8, 8), (64, 1), (65, 1), (13, 10), (51, 3), (14, 11), (16, 16), (257, 1),
         (32, 32), (41, 25)]


@pytest.mark.parametrize("wh", TILES)
@pytest.mark.parametrize("shape", [None, (64, 4, 1, 0, 3), (128, 8, 1, 0, 2), (64, 16, 1, 0, 3)])
def test_wave_tiles(rz, oracle, wh, shape):
    """Waves whose points are all on screen, over rectangles on both sides of
    every limit of the LDS tile (one pixel, one and several lanes' worth of
    entries, four, two and one copy, none): keys, sums and images."""
    cases = [dict(), dict(outside=3), dict(behind=2), dict(pile=True)]
    for i, kw in enumerate(cases):
        c, v = rectangle_scene(*wh, n=2500, seed=i, **kw)
        keys, img, sums, himg = full_render(oracle, c, v, bg=0x204060)
        pts = rz.Points.from_cloud(c)
        rz.reset_launch() if shape is None else rz.set_launch(*shape)
        try:
            fb, _ = rz.rasterize_atomicmin(pts, v, keep_keys=True, background=0x204060)
            assert np.array_equal(rz.to_u64(fb), keys), (wh, kw)
            _, acc, _, _ = rz.rasterize_hq_splat(pts, v, keep_keys=True, background=0x204060)
            assert np.array_equal(rz.unpack_acc(acc), sums), (wh, kw)
            _, _, got, st = rz.rasterize_hq_splat(pts, v, background=0x204060)
            assert np.array_equal(rz.to_u32(got), himg) and int(st.item()) == 0
            launch = None if shape is None else shape
            b = rz.Batch(pts, [v] * 3, [0, 1, 1], backgrounds=[0x204060] * 3, launch=launch)
            b.run()
            got = b.images()
            assert np.array_equal(got[0], img) and all(np.array_equal(g, himg) for g in got[1:])
        finally:
            rz.reset_launch()


@pytest.mark.parametrize("depth", [(0, 0.0), (1, 1000.0), (1, 2.0 ** 40 / 51.0),
                                   (2, ((0.0, 1e9), (2.015, 1e6), (10.0, 1e3))),
                                   (2, ((0.0, 1e9), (10.0, 1e6)))])
@pytest.mark.parametrize("eps", [(1, 100), (0, 1), (1, 3), (256, 4096), (257, 4096), (1, 4097),
                                 (1048576, 1)])
def test_wave_windows(rz, oracle, depth, eps):
    """The splat window per pixel: eps on both sides of the exact range, eps = 0,
    windows of many quanta and of less than one, piecewise maps whose ranges
    split a wave."""
    c, v = rectangle_scene(9, 7, 2000, 5)
    try:
        fbk, sums, himg = oracle.render_hq(c.x, c.y, c.z, c.rgb, v.vp, v.near, v.far, v.width,
                                           v.height, depth[0], depth[1], eps=eps)
    except Exception as e:   # the oracle refuses what the interface refuses
        with pytest.raises(rz.RzError):
            rz.rasterize_hq_splat(rz.Points.from_cloud(c), v, depth=depth, eps=eps)
        pytest.skip(f"refused by both: {e}")
    pts = rz.Points.from_cloud(c)
    fb, acc, _, _ = rz.rasterize_hq_splat(pts, v, depth=depth, eps=eps, keep_keys=True)
    assert np.array_equal(rz.to_u64(fb), fbk)
    assert np.array_equal(rz.unpack_acc(acc), sums)
    _, _, img, _ = rz.rasterize_hq_splat(pts, v, depth=depth, eps=eps)
    assert np.array_equal(rz.to_u32(img), himg)


@pytest.mark.parametrize("wh", [(1, 1), (5, 4), (8, 8), (13, 13), (14, 13), (16, 15), (22, 22),
                                (31, 32), (33, 32), (120, 90)])
@pytest.mark.parametrize("k", [2, 3, 4, 5, 7, 16])
def test_point_squares(rz, oracle, wh, k):
    """Squares of k x k pixels over rectangles of centres on both sides of every
    limit of the wave's LDS (copies, row minima, row sums), in the middle of the
    screen and against its corners: keys, sums and images."""
    for i, (kw, depth) in enumerate([(dict(), (0, 0.0)), (dict(ox=0, oy=0), (1, 1000.0)),
                                     (dict(ox=400 - wh[0], oy=300 - wh[1]), (0, 0.0)),
                                     (dict(outside=3, behind=2), (0, 0.0)), (dict(pile=True), (0, 0.0)),
                                     (dict(), (2, ((0.0, 1e9), (2.015, 1e6), (10.0, 1e3))))]):
        c, v = rectangle_scene(*wh, n=700, seed=i, **kw)
        args = (c.x, c.y, c.z, c.rgb, v.vp, v.near, v.far, v.width, v.height, *depth)
        pts = rz.Points.from_cloud(c)
        keys, img = oracle.render_atomicmin(*args, bg=7, point_size=k)
        fb, _, _, _ = rz.rasterize_points(pts, v, depth, point_size=k, background=7, keep_keys=True)
        assert np.array_equal(rz.to_u64(fb), keys), (wh, k, kw, depth)
        hk, sums, himg = oracle.render_hq(*args, bg=7, point_size=k)
        fb, acc, _, _ = rz.rasterize_points(pts, v, depth, hq=True, point_size=k, background=7,
                                            keep_keys=True)
        assert np.array_equal(rz.to_u64(fb), hk)
        assert np.array_equal(rz.unpack_acc(acc), sums), (wh, k, kw, depth)
        _, _, got, st = rz.rasterize_points(pts, v, depth, hq=True, point_size=k, background=7)
        assert np.array_equal(rz.to_u32(got), himg) and int(st.item()) == 0
    for kind in (3, 4):   # the float encodings: depth pass
        c, v = rectangle_scene(*wh, n=700, seed=9)
        keys, _ = oracle.render_atomicmin(c.x, c.y, c.z, c.rgb, v.vp, v.near, v.far, v.width,
                                          v.height, kind, 0.0, point_size=k)
        fb, _, _, _ = rz.rasterize_points(rz.Points.from_cloud(c), v, (kind, 0.0), point_size=k,
                                          keep_keys=True)
        assert np.array_equal(rz.to_u64(fb), keys)


@pytest.mark.parametrize("n", [(8 << 20) - 1, 8 << 20])
def test_batch_reads_after_clears(rz, oracle, n):
    """A batch at the size from which its flushes read nearest keys through the
    L2: replays over the same framebuffers after the cloud moved away, so that a
    key of an earlier run, were it read, would hide the points."""
    import torch
    c = gen.terrain(n, 5, extent=100.0, amplitude=10.0, wavelength=40.0)
    views = gen.orbit_views(2, 11, [(200, 150), (97, 61)], extent=100.0, rmin=60.0, rmax=120.0,
                            near=0.5, far=400.0)
    pts = rz.Points.from_cloud(c)
    b = rz.Batch(pts, views, [rz.RZ_MODE_ATOMICMIN, rz.RZ_MODE_HQ], launch=(256, 4, 1, 0, 3),
                 use_graph=True)
    scratch = torch.ones(1 << 20, device="cuda")
    for y in (c.y, c.y - np.float32(7.0), c.y - np.float32(3.0)):
        pts.y.copy_(torch.from_numpy(y))
        wants = [f(c.x, y, c.z, c.rgb, v.vp, v.near, v.far, v.width, v.height)[-1]
                 for f, v in zip((oracle.render_atomicmin, oracle.render_hq), views)]
        for _ in range(2):
            b.run()
            scratch.mul_(1.5)
            torch.cuda.synchronize()
            for got, want in zip(b.images(), wants):
                assert np.array_equal(got, want)


@pytest.mark.parametrize("k,hq", [(2, False), (3, True), (7, True)])
def test_point_squares_after_clears(rz, oracle, k, hq):
    """Frames of a cloud that moves away, into one framebuffer that each frame
    leaves cleared: a key of an earlier frame, were it read, would hide points."""
    import torch
    c = gen.terrain(300_000, 5, extent=100.0, amplitude=10.0, wavelength=40.0)
    v = gen.orbit_views(1, 11, [(200, 150)], extent=100.0, rmin=60.0, rmax=120.0, near=0.5,
                        far=400.0)[0]
    pts = rz.Points.from_cloud(c)
    fb, acc = rz.new_framebuffer(v, 0, hq=hq)
    for down in (0.0, 7.0, 3.0, 9.0):
        y = c.y - np.float32(down)
        pts.y.copy_(torch.from_numpy(y))
        render = oracle.render_hq if hq else oracle.render_atomicmin
        want = render(c.x, y, c.z, c.rgb, v.vp, v.near, v.far, v.width, v.height,
                      point_size=k)[-1]
        img = rz.rasterize_points(pts, v, hq=hq, point_size=k, fb=fb, acc=acc)[2]
        assert np.array_equal(rz.to_u32(img), want)


@pytest.mark.parametrize("n", [1, 65, (1 << 20) - 1, 1 << 20])
@pytest.mark.parametrize("depth", [(0, 0.0), (3, 0.0), (2, ((0.0, 1e9), (2.015, 1e6), (10.0, 1e3)))])
def test_small_unordered_clouds(rz, oracle, n, depth):
    """Shuffled clouds on both sides of the size from which fragments beside a tile
    read the framebuffer first, partly off screen, into a framebuffer with keys."""
    c = gen.shuffle(gen.terrain(n, 3, extent=60.0, amplitude=5.0, wavelength=20.0), 4)
    v = gen.terrain_view(120, 90, extent=50.0, distance=45.0, near=0.5, far=400.0)
    pts = rz.Points.from_cloud(c)
    keys, img = oracle.render_atomicmin(c.x, c.y, c.z, c.rgb, v.vp, v.near, v.far, v.width,
                                        v.height, *depth)
    draw = rz.rasterize_points if depth[0] == 3 else rz.rasterize_atomicmin
    fb, _ = rz.new_framebuffer(v, 0)
    for _ in range(2):   # the second time into the first one's keys
        draw(pts, v, depth, fb=fb, keep_keys=True)
        assert np.array_equal(rz.to_u64(fb), keys)
