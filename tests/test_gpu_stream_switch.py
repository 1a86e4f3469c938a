"""A context's workspace across vgicp_ctx_set_stream: a voxelization returns
while its last kernels still read the workspace on the old stream, and the
calls that use it next on another stream (a voxelization, the ordering of a
factor set's clouds) may not write it before.  The maps are those of a context
that is waited for after each call."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _cloud(rng, n, half):
    xyz = rng.uniform(-half, half, size=(n, 3)).astype(np.float32)
    xyz[:, 2] *= 0.05
    cov = np.tile(np.array([1, 0, 0, 1, 0, 1e-3], np.float32), (n, 1))
    return xyz, cov * rng.uniform(0.5, 1.5, size=(n, 1)).astype(np.float32)


def _export(m):
    return {k: v.cpu().numpy() for k, v in m.export().items()}


@pytest.mark.parametrize("then", ["voxelize", "factor_set", "grown"])
@pytest.mark.parametrize("n", [3000, 320000, (1 << 20) + 1])  # the last one is sorted
def test_next_call_on_another_stream(n, then):
    import torch
    from paper_2109_07073_amd import vgicp as vg
    rng = np.random.default_rng([n, len(then)])
    big = vg.cloud_to_device(*_cloud(rng, n, 60.0))
    # `grown` needs a larger workspace than the first call left
    small = vg.cloud_to_device(*_cloud(rng, 4 * n if then == "grown" else 20000, 40.0))
    ref_ctx = vg.Context(0)
    want = []
    for c in (big, small):
        m = vg.voxelize(ref_ctx, *c, 0.5)
        ref_ctx.synchronize()
        want.append(_export(m))
    rows = np.array([(0, 0, 0, 1)], np.int32)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    for k in range(4):
        ctx = vg.Context(0, stream=streams[k % 2])
        if then == "factor_set":
            target = vg.voxelize(ctx, *small, 0.5)
            ctx.synchronize()
        first = vg.voxelize(ctx, *big, 0.5)
        ctx.set_stream(streams[1 - k % 2])
        if then == "factor_set":
            fs = vg.FactorSet(ctx, [small], [target], rows, 2)
            assert fs.n_factors == 1
        else:
            second = vg.voxelize(ctx, *small, 0.5)
        torch.cuda.synchronize()
        got = [(first, want[0])] if then == "factor_set" else [(first, want[0]), (second, want[1])]
        for m, ref in got:
            ctx.set_stream(torch.cuda.current_stream())
            for key, v in _export(m).items():
                assert np.array_equal(v, ref[key]), (k, key)
