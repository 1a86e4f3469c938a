"""A batch's outputs are whole when its counts have arrived: a factor of more
than 16 tiles has its H written to host memory by several waves of a block,
and the server takes it as soon as the count is there.  One slot is used again
and again with other poses, so an entry that came late would be the previous
round's."""

import numpy as np
import pytest

from synth import make_tiny_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles", [17, 79])
def test_wide_batches_are_whole(tiles):
    import torch
    from paper_2109_07073_amd import vgicp as vg
    w = make_tiny_workload(seed=781, n_src=tiles * 256 - 3, n_tgt=900, resolution=0.5)
    src, tgt = w.sources[0], w.targets[0]
    ctx = vg.Context(0)
    dev = [vg.cloud_to_device(*c) for c in (src, tgt)]
    maps = [vg.voxelize(ctx, *c, 0.5) for c in dev]
    n = 96
    rows = np.array([(0, 1, 2 * k, 2 * k + 1) for k in range(n)], np.int32)
    fs = vg.FactorSet(ctx, dev, maps, rows, 2 * n, tile_points=256)
    rounds = []
    for shift in (0.0, 0.03):
        poses = np.tile(w.poses[:2], (n, 1))
        poses[:, -3:] += 0.01 * np.arange(2 * n)[:, None] + shift
        out = vg.linearize_factors(ctx, fs, torch.from_numpy(poses).to("cuda"))
        ctx.synchronize()
        rounds.append((poses, {k: v.cpu().numpy() for k, v in out.items()}))
    assert not np.array_equal(rounds[0][1]["H"], rounds[1][1]["H"])
    with vg.Server(tile_points=256, inflight=1) as srv:
        ids = [srv.add_frame(*c, 0.5) for c in (src, tgt)]
        fac = rows.copy()
        fac[:, 0], fac[:, 1] = ids
        prev = None
        for k in range(40):
            poses, ref = rounds[k % 2]
            prev = srv.submit("linearize", fac, poses, out=prev).wait()
            for key in ("H", "b", "e", "inliers"):
                assert np.array_equal(getattr(prev, key), ref[key]), (k, key)
