"""Source copies ordered by grouping against those ordered by sorting.

A cloud with more than 4,096 points in one cell is sorted instead of grouped.
Adding 5,000 points in a cell far behind every other (last in Morton order, in
no voxel) to a cloud therefore takes the other path and leaves the order of the
rest, and with it every bit of its factors, unchanged."""

import numpy as np
import pytest

from synth import make_tiny_workload
from tests.gpu_helpers import GpuWorkload, assert_linearize_parity, oracle_results

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vg():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2109_07073_amd import vgicp
    return vgicp


@pytest.fixture(scope="module")
def ctx(vg):
    return vg.Context(0)


def with_far_points(cloud, rng):
    x, c = cloud
    far = 400.0 + rng.uniform(0.05, 0.2, (5000, 3))
    return (np.concatenate([x, far.astype(np.float32)]),
            np.concatenate([c, np.tile(c[:1], (5000, 1))]))


@pytest.mark.parametrize("n,half,r", [(1, 3.0, 0.5), (255, 3.0, 0.5), (9000, 3.0, 0.5),
                                      (30000, 20.0, 0.25), (20000, 3.0, 2.0), (2000, 60.0, 0.25)])
def test_grouped_and_sorted_copies_give_the_same_bits(vg, ctx, n, half, r):
    w = make_tiny_workload(seed=800 + n, n_src=n, n_tgt=3000, resolution=r, half=half)
    a = GpuWorkload(vg, ctx, w).linearize(with_corr=True)
    w.sources = [with_far_points(w.sources[0], np.random.default_rng(n))]
    b = GpuWorkload(vg, ctx, w, tile_points=768).linearize(with_corr=True)
    for k in ("H", "b", "e", "inliers"):
        assert np.array_equal(a[k], b[k]), k
    assert np.array_equal(a["corr"], b["corr"][:n]) and np.all(b["corr"][n:] == -1)


def test_more_clouds_than_one_batch(vg, ctx):
    sizes = [1 + 7 * (k % 40) for k in range(300)]
    w = make_tiny_workload(seed=830, n_src=sizes, n_tgt=400, resolution=0.5, n_factors=len(sizes))
    w.sources[7] = (np.zeros((0, 3), np.float32), np.zeros((0, 6), np.float32))
    w.sources[9] = with_far_points(w.sources[9], np.random.default_rng(9))
    bad = w.sources[11][0].copy()
    bad[3, 1], bad[5, 0] = np.nan, np.inf
    w.sources[11] = (bad, w.sources[11][1])
    g = GpuWorkload(vg, ctx, w)
    got = g.linearize(with_corr=True)
    ref = oracle_results(w)[1]
    assert_linearize_parity(got, ref)
    assert np.array_equal(got["corr"], np.concatenate(ref["corr"]).astype(np.int32))
    assert vg.check_inputs(ctx, g.fs)["nonfinite_points"] == 2
