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
