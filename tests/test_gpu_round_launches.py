"""The launches of a round, counted as the nodes of a graph captured from it: a
round of more than 4,096 tiles writes its factors' constants in a launch of its
own only where its kernel reads them."""

import ctypes

import numpy as np
import pytest

from synth import make_tiny_workload
from tests.gpu_helpers import GpuWorkload

pytestmark = pytest.mark.gpu


def _hip():
    with open("/proc/self/maps") as f:
        path = next(line.split()[-1] for line in f if "libamdhip64" in line)
    return ctypes.CDLL(path)


def launches(hip, stream, call):
    s, graph, n = ctypes.c_void_p(stream.cuda_stream), ctypes.c_void_p(), ctypes.c_size_t()
    assert hip.hipStreamBeginCapture(s, 1) == 0  # this thread's calls only
    try:
        call()
    finally:
        assert hip.hipStreamEndCapture(s, ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    return n.value


@pytest.mark.parametrize("n_factors,table", [(2048, 0), (2049, 1)])
def test_constants_launch(n_factors, table):
    import torch
    from paper_2109_07073_amd import vgicp as vg
    hip = _hip()
    w = make_tiny_workload(seed=741, n_src=500, n_tgt=900, resolution=0.5)
    w.factors = np.tile(w.factors[:1], (n_factors, 1))
    side = torch.cuda.Stream()
    ctx = vg.Context(0, stream=side)
    g = GpuWorkload(vg, ctx, w, tile_points=256)
    assert g.fs.n_tiles == 2 * n_factors
    torch.cuda.synchronize()
    out = vg.linearize_factors(ctx, g.fs, g.poses)
    vg.linearize_factors(ctx, g.fs, g.poses, form="pair", out=out)  # allocates its partials
    torch.cuda.synchronize()
    for kw, reads in ((dict(), True), (dict(accum="f64"), True), (dict(fused="f32"), True),
                      (dict(fused="f32", fp64_kappa=100.0), False),
                      (dict(form="pair"), False), (dict(form="pair", accum="f32"), True),
                      (dict(form="pair", fused="f32"), True),
                      (dict(form="pair", fused="f32", fp64_kappa=100.0), False)):
        n = launches(hip, side, lambda: vg.linearize_factors(ctx, g.fs, g.poses, out=out, **kw))
        assert n == 2 + (table if reads else 0), kw
    cost = vg.evaluate_errors(ctx, g.fs, g.poses)
    torch.cuda.synchronize()
    assert launches(hip, side, lambda: vg.evaluate_errors(ctx, g.fs, g.poses, out=cost)) == 2 + table
