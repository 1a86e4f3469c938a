"""Replayed rounds (use_graph=True): the same bits as a plain round for new
poses in the same buffers, at one tile per factor and across the rule that
gives rounds of more than 4,096 tiles a constants launch, and refused on a
stream under capture, where a plain round is recorded."""

import numpy as np
import pytest

from synth import make_tiny_workload
from tests.gpu_helpers import GpuWorkload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_factors", [1, 1366])
def test_replay_and_capture(n_factors):
    import torch
    from paper_2109_07073_amd import vgicp as vg
    w = make_tiny_workload(seed=740, n_src=700, n_tgt=900, resolution=0.5)
    w.factors = np.tile(w.factors[:1], (n_factors, 1))
    side = torch.cuda.Stream()
    ctx = vg.Context(0, stream=side)
    g = GpuWorkload(vg, ctx, w, tile_points=256)
    assert g.fs.n_tiles == 3 * n_factors
    poses = g.poses.clone()
    torch.cuda.synchronize()
    plain = vg.linearize_factors(ctx, g.fs, poses)
    out = {k: torch.zeros_like(v) for k, v in plain.items()}
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side, capture_error_mode="thread_local"):
        with pytest.raises(vg.VgicpError):
            vg.linearize_factors(ctx, g.fs, poses, use_graph=True, out=out)
        vg.linearize_factors(ctx, g.fs, poses, out=plain)
    for rep in range(3):
        with torch.cuda.stream(side):
            poses[1, 3:] += 0.01
            vg.linearize_factors(ctx, g.fs, poses, use_graph=True, out=out)
            graph.replay()
        ctx.synchronize()
        assert int(out["inliers"][0]) > 0
        for k in out:
            assert torch.equal(out[k], plain[k]), (rep, k)
    assert g.fs.graph_count() == 1
