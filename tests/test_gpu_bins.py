"""Binning where its scan and its buffers can go wrong: bin counts around one workgroup's 2048, record buffers
that have to grow (and larger ones that are used again), and a context whose records run over several sizes.
Every frame must be bit for bit the frame of a fresh context."""
import numpy as np
import pytest

import synth
from test_gpu_parity import apc, ctx  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _scene(W, H, n_sub):
    sc = synth.scene_slabs(n_ranks=n_sub, slabs_per_rank=1, cells_per_slab=4, size=8)
    sc.view = synth.ortho_view_z(W, H)
    return sc


@pytest.mark.parametrize("sizes", [
    [(8, 8)],                                   # 4 bins
    [(256, 128)], [(248, 128)], [(264, 128)],   # 2048 bins, 64 fewer, 64 more
    [(8, 8), (300, 220), (40, 40), (512, 400)],  # grows, shrinks, grows
])
def test_frames_are_those_of_a_fresh_context(apc, sizes):
    shared = apc.Context(0)
    try:
        for W, H in sizes:
            sc = _scene(W, H, 4)
            r = apc.Renderer(shared, sc)
            r.frame(global_sum=True)
            torch.cuda.synchronize()
            mom, img = r.moments.clone(), r.rgba.clone()
            shared.resolve_pass(r.mesh, r.view, r.tf, r.mboit, r.moments, r.subs, r.rgba, finalize=True,
                                by_pair=True)  # numbers the bins that stage one made
            fresh = apc.Context(0)
            q = apc.Renderer(fresh, sc)
            q.frame(by_pair=True)  # bins, numbers and fills at once, into empty buffers
            torch.cuda.synchronize()
            assert torch.equal(q.moments, mom) and torch.equal(q.rgba, img)
            assert float((r.rgba - img).abs().max()) <= 1e-5  # the pairs' colours are grouped otherwise
            assert fresh.counters()["bin_records"] > 0
            n = fresh.moments_pass_tiles(q.mesh, q.view, q.tf, sc.m, q.subs, None, None, by_pair=True)
            # every subdomain spans the whole view: each tile with a pixel meets each of them
            assert n == -(-W // 8) * -(-H // 8) * 4
            fresh.close()
    finally:
        shared.close()
