"""Clouds at the limits of the grouped construction and of the grouped source
order, and just past them, where they are sorted instead: the same maps, the
same refusals, the same source order."""

import numpy as np
import pytest

import oracle
from synth import make_tiny_workload
from tests.gpu_helpers import GpuWorkload

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


def cloud(rng, counts, spread=60):
    """A voxel at a random place for each count, all of their points in random order."""
    at = rng.permutation(spread ** 3)[:len(counts)]
    k = np.stack([at // spread ** 2, at // spread % spread, at % spread], 1) - spread // 2
    which = rng.permutation(np.repeat(np.arange(len(counts)), counts))
    xyz = ((k[which] + rng.uniform(0.02, 0.98, (which.size, 3))) * R).astype(np.float32)
    return xyz, rng.uniform(-1, 1, (which.size, 6)).astype(np.float32)


def bricks(rng, n):
    """A point in each of n bricks, which lie apart."""
    at = rng.permutation(64 ** 3)[:n]
    k = np.stack([at // 4096, at // 64 % 64, at % 64], 1) - 32
    xyz = ((4 * k + rng.integers(0, 4, k.shape) + 0.5) * R).astype(np.float32)
    return xyz, rng.uniform(-1, 1, (n, 6)).astype(np.float32)


def check(vg, ctx, xyz, cov):
    m = vg.voxelize(ctx, *vg.cloud_to_device(xyz, cov), R)
    got = {k: v.cpu().numpy() for k, v in m.export().items()}
    ref, _ = oracle.voxelize(xyz, cov, R)
    assert np.array_equal(got["keys"], ref.keys.astype(np.int32))
    assert np.array_equal(got["count"], ref.count.astype(np.int32))
    assert np.array_equal(got["mean"], ref.mean)
    assert np.array_equal(got["cov"], ref.cov)


@pytest.mark.parametrize("counts", [
    [4097, 1, 7, 8, 9, 15, 16, 17], [5000, 4096, 4097, 64, 65] + [3] * 200, [9000]])
def test_sorted_voxels(vg, ctx, counts):
    check(vg, ctx, *cloud(np.random.default_rng(sum(counts)), counts))


@pytest.mark.parametrize("counts", [[4096] + [30] * 5000, [4097] + [30] * 5000, [64] * 2048,
                                    [64] * 2048 + [1], [64] * 8192 + [1]])
def test_points_of_several_groups_a_wave(vg, ctx, counts):
    check(vg, ctx, *cloud(np.random.default_rng(len(counts)), counts))


@pytest.mark.parametrize("n", [24000, 32768, 40000, 200000])
def test_bricks_about_the_table(vg, ctx, n):
    check(vg, ctx, *bricks(np.random.default_rng(n), n))


@pytest.mark.parametrize("kind", ["full_table", "full_voxel"])
@pytest.mark.parametrize("bad,code", [(np.nan, "ENONFINITE"), (R * 2.0 ** 20, "ERANGE")])
def test_refused_points_of_clouds_that_are_sorted(vg, ctx, kind, bad, code):
    """The refusal is the same wherever the point lies, and one call's state is
    not the next one's."""
    rng = np.random.default_rng(3)
    xyz, cov = bricks(rng, 120000) if kind == "full_table" else cloud(rng, [60000, 40])
    small = cloud(rng, [5] * 300)
    for i in (0, len(xyz) // 2, len(xyz) - 1):
        x = xyz.copy()
        x[i, 1] = bad
        with pytest.raises(vg.VgicpError) as e:
            vg.voxelize(ctx, *vg.cloud_to_device(x, cov), R)
        assert e.value.code == getattr(vg, code)
        check(vg, ctx, *small)
    both = xyz.copy()
    both[0, 0], both[-1, 0] = R * 2.0 ** 20, np.inf
    with pytest.raises(vg.VgicpError) as e:
        vg.voxelize(ctx, *vg.cloud_to_device(both, cov), R)
    assert e.value.code == vg.ENONFINITE
    check(vg, ctx, xyz, cov)


def crowded(rng, n):
    """n points in one cell."""
    return rng.uniform(0.05, 0.2, (n, 3)).astype(np.float32)


@pytest.mark.parametrize("cell,rest", [(511, 3000), (512, 3000), (513, 3000), (4000, 100),
                                       (0, 28000), (0, 90000)])
def test_source_order(vg, ctx, cell, rest):
    """As test_gpu_source_order: 5,000 more points far behind every other make a
    cloud be sorted and leave the order of the rest."""
    rng = np.random.default_rng(cell + rest)
    w = make_tiny_workload(seed=870, n_src=100, n_tgt=3000, resolution=R)
    spread = np.concatenate([w.sources[0][0], bricks(rng, rest)[0] / 2])  # half the size: 8 to a brick
    if cell == 0:
        spread = bricks(rng, rest)[0]
    xyz = np.concatenate([spread, crowded(rng, cell)])
    xyz = xyz[rng.permutation(len(xyz))]
    cov = np.tile(w.sources[0][1][:1], (len(xyz), 1)) * rng.uniform(0.5, 1.5, (len(xyz), 1))
    far = (400.0 + rng.uniform(0.05, 0.2, (5000, 3))).astype(np.float32)
    out = []
    for x, c in ((xyz, cov), (np.concatenate([xyz, far]), np.concatenate([cov, cov[:1].repeat(5000, 0)]))):
        w.sources = [(x, c.astype(np.float32))]
        out.append(GpuWorkload(vg, ctx, w, tile_points=768).linearize(with_corr=True))
    a, b = out
    for k in ("H", "b", "e", "inliers"):
        assert np.array_equal(a[k], b[k]), k
    n = len(xyz)
    assert np.array_equal(a["corr"], b["corr"][:n]) and np.all(b["corr"][n:] == -1)
