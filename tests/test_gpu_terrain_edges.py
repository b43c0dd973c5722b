"""The terrain kernels at the edges of their tiles and number ranges: normals whose quotients leave the range of the short
division (cell sizes and height differences near the ends of binary32, infinities, NaN, flat ground), streaming passes around
the 1024 texels of a block, mipmaps of every width and height modulo the 4 x 4 cells of a lane. Everything is bit-exact."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def avl():
    import paper_2506_23364_amd as m
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return m


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("cs", [1e-30, 2.0 ** -41, 2.0 ** -40, 0.3, 1.0, 10.0, 2.0 ** 39, 2.0 ** 40, 1e30])
@pytest.mark.parametrize("scale", [1e-38, 1e-20, 1e-3, 1.0, 1e10, 1e30])
def test_normals_over_the_number_range(avl, cs, scale):
    rng = np.random.default_rng(11)
    dem = (rng.standard_normal((37, 131)) * scale).astype(np.float32)
    dem[5:15, 20:90] = np.float32(scale)  # flat
    dem[20, 64:128:3] = np.inf
    dem[25, 3] = np.nan
    with np.errstate(all="ignore"):
        want = oracle.normals(dem, cs)
    got = avl.normals(dev(dem), cs).cpu().numpy()
    nan = np.isnan(want[..., :3])
    assert np.array_equal(np.isnan(got[..., :3]), nan)
    assert np.array_equal(np.where(nan, 0, got[..., :3].view(np.uint32)), np.where(nan, 0, want[..., :3].view(np.uint32)))
    np.testing.assert_allclose(got[..., 3], want[..., 3], rtol=0, atol=4e-5, equal_nan=True)


@pytest.mark.parametrize("w", [1, 255, 256, 1023, 1024, 1025, 2047, 4097])
def test_streaming_passes_at_block_edges(avl, w):
    rng = np.random.default_rng(w)
    for h in (1, 3):
        n = np.zeros((h, w, 4), np.float32)
        n[..., 2] = rng.uniform(0.3, 1.0, (h, w))
        z = rng.uniform(0, 100, (h, w)).astype(np.float32)
        z[0, ::7] = np.nan
        got = avl.snow_cover(dev(n), dev(z), 40.0, 20.0, 50.0, 15.0).cpu().numpy()
        assert np.array_equal(got.view(np.uint32), oracle.snow_cover(n, z, 40.0, 20.0, 50.0, 15.0).view(np.uint32))
        m = avl.release_mask(dev(n), dev(z), 25.0, 60.0, 10.0, 80.0).cpu().numpy()
        assert np.array_equal(m != 0, oracle.release_mask(n, z, 25.0, 60.0, 10.0, 80.0) != 0)


@pytest.mark.parametrize("h", [1, 2, 3, 4, 5, 63, 64, 66, 129])
@pytest.mark.parametrize("w", [1, 2, 3, 4, 6, 253, 255, 256, 257, 514])
def test_mipmap_of_every_remainder(avl, h, w):
    rng = np.random.default_rng(h * 1000 + w)
    c = torch.from_numpy(rng.integers(0, 1 << 32, h * w + 1).astype(np.uint32)).cuda()
    v = torch.from_numpy((rng.random(h * w + 3) * 50).astype(np.float32)).cuda()
    for oc, ov in ((0, 0), (1, 3)):  # rasters at a 16-byte boundary and off it
        ci, vi = c[oc:oc + h * w].view(h, w), v[ov:ov + h * w].view(h, w)
        ref = oracle.mipmap(ci.cpu().numpy(), vi.cpu().numpy())
        got = avl.overlay_mipmap(ci, vi)
        assert len(got) == len(ref)
        for (gc, gv), (rc, rv) in zip(got, ref):
            assert np.array_equal(gc.cpu().numpy(), rc)
            assert np.array_equal(gv.cpu().numpy(), rv)


@pytest.mark.parametrize("scale", [0.0, 3.0])
def test_normals_keep_the_sign_of_a_zero_difference(avl, scale):
    # a raster multiplied by a mask has zeros of both signs: -0.0 beside +0.0 is a difference of -0.0
    rng = np.random.default_rng(23)
    dem = (rng.standard_normal((41, 133)) * scale).astype(np.float32)
    sea = rng.random(dem.shape) < 0.7
    dem[sea] = np.where(rng.random(int(sea.sum())) < 0.5, np.float32(-0.0), np.float32(0.0))
    want = oracle.normals(dem, 10.0)
    assert np.signbit(want[want[..., 0] == 0.0][:, 0]).any() and not np.signbit(want[want[..., 0] == 0.0][:, 0]).all()
    got = avl.normals(dev(dem), 10.0).cpu().numpy()
    assert np.array_equal(got[..., :3].view(np.uint32), want[..., :3].view(np.uint32))
    both, _ = avl.normals_release_mask(dev(dem), 10.0, 30.0, 45.0, -np.inf, np.inf)
    assert np.array_equal(both.cpu().numpy().view(np.uint32), got.view(np.uint32))
