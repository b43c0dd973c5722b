"""The adjoint's sums at the edges of their tiles: particles per cell around the 16 and 64 of a transposed load, release cells
around a wave's 16 and a block's 64, particles around the 4096 of a block's chunk. The per-particle terms are the kernel's
own (checked against the oracle elsewhere); their sums in order, in binary64, give dL/dmass bit for bit."""
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


@pytest.mark.parametrize("n_cells,P", [(1, 1), (1, 64), (15, 16), (16, 15), (17, 17), (63, 65), (64, 64), (65, 63), (64, 129),
                                       (130, 127), (4096, 1), (4097, 1), (257, 16), (1, 4097)])
def test_sums_in_order(avl, n_cells, P):
    dem = synth.incline_fillet_dem(160, 10.0, seed=6)
    mask = np.zeros(dem.shape, np.uint8)
    mask.reshape(-1)[np.random.default_rng(P).permutation(dem.size // 2)[:n_cells]] = 1
    rng = np.random.default_rng(n_cells)
    d, m = torch.from_numpy(dem).cuda(), torch.from_numpy(mask).cuda()
    g = torch.from_numpy(rng.standard_normal(dem.shape).astype(np.float32)).cuda()
    par = avl.Params.make(**dict(synth.DEFAULT_PARAMS, mu=0.25, xi=1500.0, randomness=0.3))
    for cap in (n_cells, 3 * n_cells + 70):  # sums sized for the capacity, not the cells that are there
        r = avl.trajectories_smooth(d, m, 10.0, par, P, 500, 3, max_release_cells=cap)
        dp, dm, pp = (x.cpu().numpy() for x in avl.trajectories_backward(r, d, m, 10.0, par, P, 500, 3, g,
                                                                         per_particle=True))
        n = n_cells * P
        pp = pp[:, :n].astype(np.float64)
        want = (np.cumsum(pp[3].reshape(n_cells, P), axis=1)[:, -1] / P).astype(np.float32)
        assert np.array_equal(dm.reshape(-1)[np.flatnonzero(mask)], want)
        assert not dm.reshape(-1)[np.flatnonzero(mask == 0)].any()
        # any order of n binary64 additions is within n ulps of the sum of magnitudes
        for k in range(3):
            assert abs(dp[k] - pp[k].sum()) <= 2.0 * n * 2.0 ** -53 * np.abs(pp[k]).sum()


@pytest.mark.parametrize("n_cells,P,limit", [(1, 1, 500), (3, 85, 500), (1, 257, 500), (2, 1025, 500), (300, 7, 64), (300, 7, 65),
                                             (200, 10, 3), (200, 10, 0),
                                             (3100, 260, 3)])
def test_adjoint_windows(avl, n_cells, P, limit):
    """Every window size gives the oracle's terms: particles around a window's and a wave's, paths that end at the release, in
    the first segment, at a checkpoint and segments later, more or fewer steps than are kept in LDS, exits and limits;
    one window a block and (806,000 particles) several."""
    import oracle
    dem = synth.incline_fillet_dem(160, 10.0, seed=6)
    mask = np.zeros(dem.shape, np.uint8)
    mask.reshape(-1)[np.random.default_rng(P).permutation(dem.size // 2)[:n_cells]] = 1
    rng = np.random.default_rng(n_cells)
    gD = rng.standard_normal(dem.shape).astype(np.float32)
    p = dict(synth.DEFAULT_PARAMS, mu=0.25, xi=1500.0, randomness=0.3)
    want = oracle.smooth_backward(dem, mask, 10.0, oracle.make_params(**p), P, limit, 3, gD).per_particle
    d, m, g = (torch.from_numpy(x).cuda() for x in (dem, mask, gD))
    par = avl.Params.make(**p)
    try:
        for v in range(avl.smooth_tuning_variants()[1]):
            avl.set_smooth_tuning(-1, v)
            r = avl.trajectories_smooth(d, m, 10.0, par, P, limit, 3)
            pp = avl.trajectories_backward(r, d, m, 10.0, par, P, limit, 3, g, per_particle=True)[2].cpu().numpy()
            assert np.array_equal(pp[:, :n_cells * P].T, want), f"variant {v}"
    finally:
        avl.set_smooth_tuning(-1, -1)
