"""A calibration whose capacity is far above its release: most blocks of the iteration's sums hold no particles, and may start
after the last one that does has set up the next iteration's run. History and result are those of the tight capacity, bit
for bit, and an iterate that leaves the parameters' range is reported with its iteration."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def avl():
    import paper_2506_23364_amd as m
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return m


def scene():
    dem = synth.alpine_dem(128, 700.0, seed=4)[:120, :113].copy()
    mask = np.zeros(dem.shape, np.uint8)
    mask[20:26, 30:41] = 1
    target = np.zeros(dem.shape, np.float32)
    target[30:40, 35:50] = 0.4
    return [torch.from_numpy(a).cuda() for a in (dem, mask, target)]


@pytest.mark.parametrize("P", [1, 33])
def test_surplus_capacity_changes_nothing(avl, P):
    dem, mask, target = scene()
    start = avl.Params.make(mu=0.2, xi=1500.0)
    n = int(mask.sum())
    ref, rp = avl.calibrate(dem, mask, 10.0, start, P, 400, 7, target, 12, max_release_cells=n)
    for cap in (n + 1, mask.numel()):
        hist, p = avl.calibrate(dem, mask, 10.0, start, P, 400, 7, target, 12, max_release_cells=cap)
        assert np.array_equal(hist, ref) and p.mu == rp.mu and p.xi == rp.xi
    assert ref[0, 0] > 0.0 and len(np.unique(ref[:, 1])) == 12


def test_an_iterate_out_of_range_is_reported(avl):
    # the release itself as target: more friction brings the deposit nearer, so the first step moves mu up by 3e38, the second
    # past binary32's largest number: iteration 2 has no valid parameters
    dem, mask, _ = scene()
    adam = avl.Adam.make(lr_mu=3e38)
    start = avl.Params.make(mu=0.2, xi=1500.0)
    for cap in (int(mask.sum()), mask.numel()):
        hist, _ = avl.calibrate(dem, mask, 10.0, start, 4, 400, 7, mask.float(), 2, adam, max_release_cells=cap)
        assert hist[0, 3] < 0.0 and hist[1, 1] > 2e38
        with pytest.raises(avl.AvlError, match="iteration 2"):
            avl.calibrate(dem, mask, 10.0, start, 4, 400, 7, mask.float(), 6, adam, max_release_cells=cap)
