"""The preparation kernels at the edges of their chunks: release-cell lists around 4096 texels per block, 16 bytes per
thread and the number of blocks up to which no scan of the counts runs; padded DEMs narrower than one 16-byte store;
ensembles whose tiles start at unaligned addresses."""
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


@pytest.mark.parametrize("shape", [(1, 1), (1, 15), (3, 5), (1, 4095), (64, 64), (17, 241), (241, 17), (2048, 4096),
                                   (2049, 4096), (2897, 2897)])
@pytest.mark.parametrize("density", [0.0, 0.02, 1.0])
def test_release_cells_at_chunk_edges(avl, shape, density):
    rng = np.random.default_rng(shape[0] * 7 + shape[1])
    m = (rng.random(shape) < density).astype(np.uint8) * 255
    cells, n = avl.release_cells(torch.from_numpy(m).cuda())
    want = np.flatnonzero(m)
    assert int(n.item()) == want.size
    assert np.array_equal(cells[:want.size].cpu().numpy(), want)


@pytest.mark.parametrize("shape", [(1, 1), (5, 1), (4, 2), (3, 3), (9, 4), (7, 5), (6, 7), (33, 31)])
def test_narrow_grids(avl, shape):
    rng = np.random.default_rng(shape[0] * 11 + shape[1])
    dem = (rng.random(shape) * 20.0).astype(np.float32)
    mask = np.ones(shape, np.uint8)
    p = dict(synth.DEFAULT_PARAMS, mu=0.1)
    ref = oracle.trajectories(dem, mask, 5.0, oracle.make_params(**p), 3, 60, 9)
    got = avl.trajectories(torch.from_numpy(dem).cuda(), torch.from_numpy(mask).cuda(), 5.0, avl.Params.make(**p), 3, 60, 9)
    assert np.array_equal(got.counts.cpu().numpy(), ref.counts)
    np.testing.assert_allclose(got.vmax.cpu().numpy(), ref.vmax, rtol=1e-5, atol=0)
    assert list(got.stats.cpu().numpy()) == [ref.steps, ref.n_exit, ref.n_stop, ref.n_limit]


def test_batch_of_odd_tiles(avl):
    rng = np.random.default_rng(3)
    dems = (rng.random((3, 13, 11)) * 30.0).astype(np.float32)
    masks = (rng.random((2, 13, 11)) < 0.4).astype(np.uint8)
    p = dict(synth.DEFAULT_PARAMS, mu=0.1)
    runs = [(t, s, 0, 5 * t + s, 77) for t in range(3) for s in range(2)]
    r = avl.trajectories_batched(torch.from_numpy(dems).cuda(), torch.from_numpy(masks).cuda(), 5.0,
                                 avl.params_tensor([p], "cuda"), avl.runs_tensor(runs, "cuda"), 4, 80)
    for k, (t, s, _, run_id, seed) in enumerate(runs):
        ref = oracle.trajectories(dems[t], masks[s], 5.0, oracle.make_params(**p), 4, 80, seed, run_id)
        assert np.array_equal(r.counts[k].cpu().numpy(), ref.counts), k
        np.testing.assert_allclose(r.vmax[k].cpu().numpy(), ref.vmax, rtol=1e-5, atol=0)


def test_batch_of_more_small_tiles_than_one_launch_holds(avl):
    # a block per tile and per mask: 2^24 blocks of 256 threads would be 2^32 threads
    n = (1 << 24) + 5
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    dems = torch.rand(n, 2, 2, device="cuda", generator=g) * 30.0
    masks = (torch.rand(n, 2, 2, device="cuda", generator=g) < 0.5).to(torch.uint8)
    p = dict(synth.DEFAULT_PARAMS, mu=0.1)
    at = [0, 1, (1 << 23) - 1, 1 << 23, (1 << 24) - 1, 1 << 24, n - 1]
    runs = [(t, at[-1 - k], 0, k, 7) for k, t in enumerate(at)]
    r = avl.trajectories_batched(dems, masks, 5.0, avl.params_tensor([p], "cuda"), avl.runs_tensor(runs, "cuda"), 3, 40)
    for k, (t, s, _, run_id, seed) in enumerate(runs):
        ref = oracle.trajectories(dems[t].cpu().numpy(), masks[s].cpu().numpy(), 5.0, oracle.make_params(**p), 3, 40, seed, run_id)
        assert np.array_equal(r.counts[k].cpu().numpy(), ref.counts), k
        assert list(r.stats[k].cpu().numpy()) == [ref.steps, ref.n_exit, ref.n_stop, ref.n_limit], k
    del dems, masks, r
    torch.cuda.empty_cache()


@pytest.mark.parametrize("shape,n_masks", [((2897, 2897), 2), ((2048, 4096), 2), ((1024, 1028), 63),
                                           ((1024, 1028), 64), ((512, 2048), 66)])
def test_batch_of_large_sparse_masks(avl, shape, n_masks):
    # several masks with and without a scan of their counts: a run of each equals the plain call
    rng = np.random.default_rng(n_masks)
    dem = torch.from_numpy((rng.random(shape) * 15.0).astype(np.float32)).cuda()[None]
    masks = torch.zeros((n_masks, *shape), dtype=torch.uint8, device="cuda")
    for s in range(n_masks):  # few cells, first and last texel of every third mask among them
        at = np.concatenate([rng.integers(0, dem.numel(), 40 + s), [0, dem.numel() - 1] if s % 3 == 0 else []]).astype(np.int64)
        masks[s].view(-1)[torch.from_numpy(at).cuda()] = 1
    p = dict(synth.DEFAULT_PARAMS, mu=0.1)
    used = [0, 1, n_masks // 2, n_masks - 1]
    r = avl.trajectories_batched(dem, masks, 5.0, avl.params_tensor([p], "cuda"),
                                 avl.runs_tensor([(0, s, 0, k, 19) for k, s in enumerate(used)], "cuda"), 5, 60)
    for k, s in enumerate(used):
        one = avl.trajectories(dem[0], masks[s], 5.0, avl.Params.make(**p), 5, 60, 19, run_id=k)
        assert int(one.counts.view(torch.int32).sum()) > 0
        assert torch.equal(r.counts[k].view(torch.int32), one.counts.view(torch.int32)), s
        assert torch.equal(r.vmax[k], one.vmax), s
        assert torch.equal(r.stats[k].view(torch.int64), one.stats.view(torch.int64)), s
