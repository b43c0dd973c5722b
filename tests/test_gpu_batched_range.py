"""Speeds of a batch over the number range: tiles whose squared speeds fall below 2^-96 and to subnormals, ordinary ones, and
ones where they overflow, together in one batch, so that waves flush odd and ordinary roots side by side. Every run's rasters
equal those of the single-run call, which takes its roots in a pass of its own, bit for bit and on every kernel variant."""
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


@pytest.mark.parametrize("density", [0.02, 1.0])
def test_batch_speeds_over_the_number_range(avl, density):
    rng = np.random.default_rng(31)
    h, w = 48, 40
    base = rng.random((h, w))
    dems = np.stack([(base * s).astype(np.float32) for s in (1e-16, 1e-22, 1e-30, 1e-36, 1e-41, 25.0, 1e17, 1e30, 3e38)])
    masks = (rng.random((2, h, w)) < density).astype(np.uint8)
    params = [dict(synth.DEFAULT_PARAMS, mu=0.0, xi=float("inf"), randomness=0.2), dict(synth.DEFAULT_PARAMS, mu=0.0, xi=900.0)]
    n = len(dems)
    # neighbouring runs on tiles of different scales
    runs = [(t, s, q, 3 * t + s, 11) for q in range(2) for s in range(2) for t in range(n)]
    d, m = torch.from_numpy(dems).cuda(), torch.from_numpy(masks).cuda()
    want = [avl.trajectories(d[t], m[s], 10.0, avl.Params.make(**params[q]), 6, 50, seed, run_id=rid) for t, s, q, rid, seed in runs]
    got_small = got_odd = 0
    try:
        for v in range(avl.tuning_variants()):
            avl.set_tuning(v, True)
            r = avl.trajectories_batched(d, m, 10.0, avl.params_tensor(params, "cuda"), avl.runs_tensor(runs, "cuda"), 6, 50)
            for k, ref in enumerate(want):
                assert torch.equal(r.counts[k].view(torch.int32), ref.counts.view(torch.int32)), (v, k)
                assert torch.equal(r.stats[k].view(torch.int64), ref.stats.view(torch.int64)), (v, k)
                a, b = r.vmax[k], ref.vmax
                nan = b.isnan()
                assert torch.equal(a.isnan(), nan), (v, k)
                assert torch.equal(a[~nan].view(torch.int32), b[~nan].view(torch.int32)), (v, k)
                got_small += int(((b > 0) & (b < 2.0 ** -48)).sum())
                got_odd += int((~b.isfinite()).sum())
    finally:
        avl.set_tuning(-1, True)
    assert got_small > 0 and got_odd > 0
