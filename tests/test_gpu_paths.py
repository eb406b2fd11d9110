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
