"""The velocity raster, through its table and (few particles) straight: every forward variant, releases close together (cells shared, several flushes) and scattered
(buckets overflow to the raster), masses whose fixed point needs 64 bits, one and several slots per lane."""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def avl():
    import paper_2506_23364_amd as m
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return m


@pytest.mark.parametrize("density,P,mass_scale", [(0.02, 40, 1.0), (0.3, 1, 1.0), (0.05, 3, 5000.0), (0.001, 1, 1.0),
                                                  (0.002, 17, 3000.0), (0.05, 17, 5000.0)])
def test_velocity_raster_every_variant(avl, density, P, mass_scale):
    dem = synth.incline_fillet_dem(160, 10.0, seed=5)[:, :131].copy()
    rng = np.random.default_rng(8)
    mask = ((rng.random(dem.shape) < density) & (np.arange(160)[:, None] < 60)).astype(np.uint8)
    mass = (rng.uniform(0.5, 1.5, dem.shape) * mass_scale).astype(np.float32)
    p = dict(synth.DEFAULT_PARAMS, mu=0.25, xi=1500.0, randomness=0.3)
    ref = oracle.smooth_forward(dem, mask, 10.0, oracle.make_params(**p), P, 700, 21, mass=mass, vel_splat=True)
    d, m, ms = (torch.from_numpy(a).cuda() for a in (dem, mask, mass))
    try:
        for v in range(avl.smooth_tuning_variants()[0]):
            avl.set_smooth_tuning(v, -1)
            r = avl.trajectories_smooth(d, m, 10.0, avl.Params.make(**p), P, 700, 21, mass=ms, velocity=True)
            assert np.array_equal(r.deposit_q.cpu().numpy(), ref.dep_q), f"variant {v}"
            assert np.array_equal(r.velocity_q.cpu().numpy(), ref.vel_q), f"variant {v}"
            assert list(r.stats.cpu().numpy()) == [ref.steps, ref.n_exit, ref.n_stop, ref.n_limit], f"variant {v}"
            assert np.array_equal(r.velocity.cpu().numpy(), (ref.vel_q * 2.0 ** -24).astype(np.float32)), f"variant {v}"
    finally:
        avl.set_smooth_tuning(-1, -1)


@pytest.mark.parametrize("P", [8, 9, 16])
@pytest.mark.parametrize("reach", [0, 128, 1024])
@pytest.mark.parametrize("over", [0, 1])
def test_velocity_raster_at_the_limits_of_its_two_forms(avl, P, reach, over):
    # releases at, and one cell past, 3072 particles and reach 3072 / P^2 of them
    cells = (3072 if reach == 0 else reach * 3072 // P ** 2) // P + over
    dem = synth.alpine_dem(256, 1000.0, seed=12)[:250, :211].copy()
    mask = np.zeros(dem.size, np.uint8)
    mask[np.random.default_rng(6).permutation(dem.size)[:max(1, cells)]] = 1
    mask = mask.reshape(dem.shape)
    p = dict(synth.DEFAULT_PARAMS, mu=0.25, xi=1500.0)
    ref = oracle.smooth_forward(dem, mask, 10.0, oracle.make_params(**p), P, 300, 33, vel_splat=True)
    d, m = (torch.from_numpy(a).cuda() for a in (dem, mask))
    n = avl.smooth_tuning_variants()[0]
    try:
        for v in (-1, 0, n // 2, n - 1):  # the tuner's choice, the first shape without and with a straight start, the last with
            avl.set_smooth_tuning(v, -1)
            r = avl.trajectories_smooth(d, m, 10.0, avl.Params.make(**p), P, 300, 33, velocity=True)
            assert np.array_equal(r.velocity_q.cpu().numpy(), ref.vel_q), f"variant {v}"
            assert np.array_equal(r.deposit_q.cpu().numpy(), ref.dep_q), f"variant {v}"
    finally:
        avl.set_smooth_tuning(-1, -1)
