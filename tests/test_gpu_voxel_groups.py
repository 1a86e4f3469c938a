"""Voxel maps at the edges of the grouped construction, bit for bit against the
oracle: voxels of as many points as one wave, one gather, one sorted list and
the whole path take; clouds of few points, of the largest grouped size and one
more; clouds whose bricks do not fit its table; and points it refuses."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

R = 0.5


@pytest.fixture(scope="module")
def vg():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2109_07073_amd import vgicp
    return vgicp


@pytest.fixture(scope="module")
def ctx(vg):
    return vg.Context(0)


def check(vg, ctx, xyz, cov):
    m = vg.voxelize(ctx, *vg.cloud_to_device(xyz, cov), R)
    got = {k: v.cpu().numpy() for k, v in m.export().items()}
    ref, inv = oracle.voxelize(xyz, cov, R)
    assert np.array_equal(got["keys"], ref.keys.astype(np.int32))
    assert np.array_equal(got["count"], ref.count.astype(np.int32))
    assert np.array_equal(got["mean"], ref.mean)
    assert np.array_equal(got["cov"], ref.cov)
    # every point finds its own voxel through the brick table
    fs = vg.FactorSet(ctx, [vg.cloud_to_device(xyz, cov)], [m], [(0, 0, 0, 0)], 1)
    import torch
    pose = torch.tensor([[1, 0, 0, 0, 1, 0, 0, 0, 1, 0, 0, 0]], dtype=torch.float64, device="cuda")
    corr = vg.linearize_factors(ctx, fs, pose, with_corr=True)["corr"]
    ctx.synchronize()
    assert np.array_equal(corr.cpu().numpy(), inv.astype(np.int32))


def cloud(rng, counts, spread):
    """A voxel at a random place for each count, its points in random order among the others'."""
    at = rng.permutation(spread ** 3)[:len(counts)]
    k = np.stack([at // spread ** 2, at // spread % spread, at % spread], 1) - spread // 2
    which = rng.permutation(np.repeat(np.arange(len(counts)), counts))
    xyz = ((k[which] + rng.uniform(0.02, 0.98, (which.size, 3))) * R).astype(np.float32)
    return xyz, rng.uniform(-1, 1, (which.size, 6)).astype(np.float32)


@pytest.mark.parametrize("counts", [
    [1], [63], [64, 1], [65], [255, 256], [257, 2], [512, 513], [4096], [4097],
    [1] * 300, [64] * 40 + [65] * 40, list(range(1, 140))])
def test_points_per_voxel(vg, ctx, counts):
    rng = np.random.default_rng(sum(counts))
    check(vg, ctx, *cloud(rng, counts, 9))


@pytest.mark.parametrize("n", [(1 << 20), (1 << 20) + 1])
def test_largest_grouped_cloud(vg, ctx, n):
    rng = np.random.default_rng(n)
    xyz = rng.uniform([-30, -30, -2], [30, 30, 2], (n, 3)).astype(np.float32)
    check(vg, ctx, xyz, rng.uniform(-1, 1, (n, 6)).astype(np.float32))


@pytest.mark.parametrize("n", [300, 5000, 30000])
def test_a_brick_for_every_point(vg, ctx, n):
    rng = np.random.default_rng(n)
    check(vg, ctx, *cloud(rng, [1] * n, 400))


@pytest.mark.parametrize("bad,code", [(np.nan, "ENONFINITE"), (np.inf, "ENONFINITE"),
                                      (R * 2.0 ** 20, "ERANGE"), (-R * 2.0 ** 20 - 1, "ERANGE")])
def test_refused_points(vg, ctx, bad, code):
    rng = np.random.default_rng(5)
    xyz, cov = cloud(rng, [3] * 100, 9)
    for i, a in ((0, 0), (150, 1), (299, 2)):
        x = xyz.copy()
        x[i, a] = bad
        with pytest.raises(vg.VgicpError) as e:
            vg.voxelize(ctx, *vg.cloud_to_device(x, cov), R)
        assert e.value.code == getattr(vg, code)
    check(vg, ctx, xyz, cov)


def test_first_map_of_each_context(vg):
    """Each context's first map has its own counts, also where its pinned words
    last held an earlier context's first counts."""
    rng = np.random.default_rng(9)
    for counts in ([3] * 2000, [1], [2] * 500, [64] * 3, [1] * 4000, [5]):
        own = vg.Context(0)
        check(vg, own, *cloud(rng, counts, 30))
        own.close()


def test_lookups_past_bricks_at_minus_one(vg, ctx):
    """Bricks with y = z = -1, whose record keys have all ones in their low
    half, are home records that lookups of other bricks probe past."""
    rng = np.random.default_rng(11)
    x = np.arange(-4000, 4000)
    bricks = np.concatenate([np.stack([x, np.full_like(x, -1), np.full_like(x, -1)], 1),
                             rng.integers(-300, 300, (8000, 3))])
    xyz = ((4 * bricks + rng.integers(0, 4, bricks.shape) + 0.5) * R).astype(np.float32)
    check(vg, ctx, xyz, rng.uniform(-1, 1, (len(xyz), 6)).astype(np.float32))
