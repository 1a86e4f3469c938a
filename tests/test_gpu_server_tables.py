"""A server batch's tables and outputs at their edges: tiles of a factor made 64
at a time, descriptors and poses on either side of a wave, factors without
points, each kind in both variants of the reduce.  The bits are those of a
factor set with the server's tile size."""

import numpy as np
import pytest

from synth import make_tiny_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_src", [0, 1, 256, 257, 64 * 256, 65 * 256 + 3])
@pytest.mark.parametrize("n_factors", [1, 64, 65])
def test_batch_matches_factor_set(n_src, n_factors):
    import torch
    from paper_2109_07073_amd import vgicp as vg
    w = make_tiny_workload(seed=760, n_src=max(n_src, 1), n_tgt=900, resolution=0.5)
    (xyz, cov), tgt = w.sources[0], w.targets[0]
    src = (xyz[:n_src], cov[:n_src])
    ctx = vg.Context(0)
    dev = [vg.cloud_to_device(*c) for c in (src, tgt)]
    maps = [vg.voxelize(ctx, *c, 0.5) for c in dev]
    rows = np.array([(k % 2, 1, 2 * k, 2 * k + 1) for k in range(n_factors)], np.int32)
    poses = np.tile(w.poses[:2], (n_factors, 1))
    poses[:, -3:] += 0.01 * np.arange(2 * n_factors)[:, None]
    fs = vg.FactorSet(ctx, dev, maps, rows, 2 * n_factors, tile_points=256)
    d_poses = torch.from_numpy(poses).to("cuda")
    lin = vg.linearize_factors(ctx, fs, d_poses)
    cost = vg.evaluate_errors(ctx, fs, d_poses)
    over = vg.overlap(ctx, fs, d_poses)
    ctx.synchronize()
    assert n_src < 256 or int(lin["inliers"].sum()) > 0
    with vg.Server(tile_points=256) as srv:
        ids = [srv.add_frame(*c, 0.5) for c in (src, tgt)]
        fac = rows.copy()
        fac[:, 0] = [ids[s] for s in rows[:, 0]]
        fac[:, 1] = ids[1]
        for kind, ref, keys in (("linearize", lin, ("H", "b", "e", "inliers")),
                                ("evaluate", cost, ("e", "inliers"))):
            got = srv.submit(kind, fac, poses).wait()
            for k in keys:
                assert np.array_equal(getattr(got, k), ref[k].cpu().numpy()), (kind, k)
        got = srv.submit("overlap", fac, poses).wait()
        assert np.array_equal(got.inliers, over["hits"].cpu().numpy())
        assert np.array_equal(got.overlap, over["overlap"].cpu().numpy())
