"""Frames on a stream that the caller captures in a graph of its own: a frame whose bins are at hand launches kernels
only, and its replays are bit for bit the eager frame; whatever has to read its totals back is refused, with the
capture still whole and nothing launched."""
import pytest

import synth
from test_gpu_parity import apc  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture()
def frame(apc):
    own = apc.Context(0)
    sc = synth.scene_tiny()
    r = apc.Renderer(own, sc)
    yield own, r, sc
    own.close()


def test_what_reads_totals_back_is_refused(apc, frame):
    ctx, r, sc = frame
    graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    r.frame(global_sum=True)  # sizes the buffers, bins and numbers this view
    torch.cuda.synchronize()
    other = apc.make_view(synth.ortho_view_z(120, 100), sc.step)
    mom = torch.zeros((sc.m + 1, 100, 120), device="cuda")
    rgba = torch.zeros((100, 120, 4), device="cuda")
    n = ctx.counters()["bin_records"]
    with torch.cuda.graph(graph, stream=stream):
        s = stream.cuda_stream
        for call in (
            lambda: ctx.moments_pass(r.mesh, other, r.tf, sc.m, r.subs, mom, s, global_sum=True),
            lambda: ctx.resolve_pass(r.mesh, other, r.tf, r.mboit, mom, r.subs, rgba, stream=s),
            lambda: ctx.resolve_pass_noalloc(r.mesh, other, r.tf, r.mboit, mom, r.subs, rgba, stream=s),
            lambda: ctx.resolve_pass(r.mesh, r.view, r.tf, r.mboit, r.moments, r.subs, r.rgba, stream=s, by_pair=True),
            lambda: ctx.moments_pass_tiles(r.mesh, r.view, r.tf, sc.m, r.subs, stream=s, by_pair=True),
        ):
            with pytest.raises(apc.ApcError):
                call()
        mom.zero_()  # (a graph with a node)
    torch.cuda.synchronize()
    assert ctx.counters()["bin_records"] == n


@pytest.mark.parametrize("first", ["moments", "kept", "resolve"])
def test_replays_of_a_captured_frame_are_the_eager_frame(apc, frame, first):
    """Whatever made the bins: with numbered pairs stage one goes by pairs, else per tile, the same bits."""
    ctx, r, sc = frame
    want = r.frame(global_sum=True).clone()
    mom = r.moments.clone()
    ctx.set_dispatch(apc.APC_DISPATCH_QUEUE)  # sizes the per-tile form's buffers
    r.frame(global_sum=True)
    ctx.set_dispatch(apc.APC_DISPATCH_GRID)
    elsewhere = synth.ortho_view_z(*[r.view.width, r.view.height])
    elsewhere["eye"] = tuple(e + d for e, d in zip(elsewhere["eye"], (1e-3, 0.0, 0.0)))
    other = apc.make_view(elsewhere, sc.step)
    ctx.resolve_pass(r.mesh, other, r.tf, r.mboit, r.moments, r.subs, r.rgba)  # other bins
    if first == "resolve":
        ctx.resolve_pass(r.mesh, r.view, r.tf, r.mboit, r.moments, r.subs, r.rgba)
    else:
        ctx.moments_pass(r.mesh, r.view, r.tf, sc.m, r.subs, r.moments, keep=first == "kept", global_sum=True)
    torch.cuda.synchronize()
    graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=stream):
        s = stream.cuda_stream
        ctx.moments_pass(r.mesh, r.view, r.tf, sc.m, r.subs, r.moments, s, global_sum=True)
        ctx.resolve_pass(r.mesh, r.view, r.tf, r.mboit, r.moments, r.subs, r.rgba, stream=s)
    for _ in range(3):
        r.moments.fill_(-1.0)
        r.rgba.fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(r.moments, mom) and torch.equal(r.rgba, want)
