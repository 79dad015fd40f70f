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


@pytest.mark.parametrize("W,H,n_sub,m", [
    (1, 1, 1, 4), (61, 43, 5, 8), (200, 120, 16, 6),
    (1024, 1024, 2, 4),    # 16384 tiles, the most that go by pairs; 32768 pairs of 1280 bytes
    (1025, 1024, 2, 4),    # a column of tiles more: per tile
    (1024, 1024, 16, 8),   # 262144 pairs, 604 MB of moments: per tile
])
def test_stage_one_of_few_tiles_by_pairs_is_the_per_tile_pass(apc, ctx, W, H, n_sub, m):
    """A work queue takes whole tiles, the grid of a frame of few tiles (tile, subdomain) pairs: the same moments,
    per subdomain and global, segment counts, images and counters, bit for bit; also for a subset in another
    order."""
    sc = _scene(W, H, n_sub)
    sc.view = synth.perspective_view((0.5, 2.3, 0.9), (0.5, 0.5, 0.5), W, H)  # some tiles meet few subdomains
    sc.m, sc.bias = m, synth.default_bias(m)
    r = apc.Renderer(ctx, sc)
    part = np.asarray([n_sub - 1] + list(range(0, n_sub - 1, 2)), np.int32)
    got = {}
    try:
        for mode in (apc.APC_DISPATCH_QUEUE, apc.APC_DISPATCH_GRID):
            ctx.set_dispatch(mode)
            out = []
            for kw in (dict(global_sum=True), dict(), dict(subdomains=part)):
                ctx.counters(reset=True)
                r.moments.fill_(-1.0)
                r.per_sub.fill_(-1.0)
                img = r.frame(**kw).clone()
                c = ctx.counters()
                out += [img, r.moments.clone(), r.per_sub.clone(), ctx.segment_counts(H, W),
                        torch.tensor([c[k] for k in ("pieces", "tet_steps", "entries", "segments", "nonpd_pivots")])]
            got[mode] = out
    finally:
        ctx.set_dispatch(apc.APC_DISPATCH_GRID)
    for k, (a, b) in enumerate(zip(*got.values())):
        assert torch.equal(a, b), k


def test_images_beyond_one_row_of_the_clearing_launch(apc, ctx):
    """Per-subdomain images of more than 2^28 values (the clearing's grid then has rows): bit for bit the per-tile
    pass's, zeros where no pair writes included."""
    n_sub, W, H, m = 31, 1024, 1024, 8
    sc = _scene(W, H, n_sub)
    sc.view = synth.perspective_view((0.5, 2.3, 0.9), (0.5, 0.5, 0.5), W, H)
    sc.m, sc.bias = m, synth.default_bias(m)
    r = apc.Renderer(ctx, sc)
    assert r.per_sub.numel() > 1 << 28
    got = []
    try:
        for mode in (apc.APC_DISPATCH_QUEUE, apc.APC_DISPATCH_GRID):
            ctx.set_dispatch(mode)
            r.per_sub.fill_(-1.0)
            ctx.moments_pass(r.mesh, r.view, r.tf, m, r.subs, r.per_sub)
            torch.cuda.synchronize()
            got.append(r.per_sub.clone())
    finally:
        ctx.set_dispatch(apc.APC_DISPATCH_GRID)
    assert torch.equal(*got)


@pytest.mark.parametrize("W,H,n_sub,pairs", [
    (512, 288, 1, False), (392, 384, 1, True), (768, 768, 1, True), (776, 768, 1, False),
    (8, 8, 2, True), (768, 768, 3, True), (776, 768, 3, False), (1000, 1000, 8, True), (1032, 1024, 8, False),
])
def test_both_forms_of_stage_one_on_both_sides_of_the_line(apc, W, H, n_sub, pairs):
    """Frames on both sides of the lines between the forms: the expected form ran (the per-tile one of a global sum
    needs its FP64 partials, which a context that went by pairs gets only for the work queue's frame after it), and
    moments, images per subdomain and segment counts are the queue's bit for bit."""
    sc = _scene(W, H, n_sub)
    sc.view = synth.perspective_view((0.5, 2.3, 0.9), (0.5, 0.5, 0.5), W, H)
    sc.m, sc.bias = 4, synth.default_bias(4)
    own = apc.Context(0)
    try:
        r = apc.Renderer(own, sc)
        got = []
        for mode in (apc.APC_DISPATCH_GRID, apc.APC_DISPATCH_QUEUE):
            own.set_dispatch(mode)
            before = own.workspace_bytes()
            r.moments.fill_(-1.0)
            own.moments_pass(r.mesh, r.view, r.tf, sc.m, r.subs, r.moments, global_sum=True)
            grown = own.workspace_bytes() - before
            seg = own.segment_counts(H, W)
            r.per_sub.fill_(-1.0)
            own.moments_pass(r.mesh, r.view, r.tf, sc.m, r.subs, r.per_sub)
            got.append([r.moments.clone(), seg, r.per_sub.clone(), own.segment_counts(H, W)])
        assert (grown >= 8 * 5 * W * H) == pairs
        for a, b in zip(*got):
            assert torch.equal(a, b)
    finally:
        own.close()


@pytest.mark.parametrize("size,n_sub", [(1024, 36), (4096, 64), (4096, 72)])
def test_numbers_and_offsets_of_millions_of_bins(apc, ctx, size, n_sub):
    """589,824, 16.8 and 18.9 million bins (more workgroups of the scan than one has threads; the last with its sums
    in two levels): the list of the pairs is exactly that of the subdomains binned one at a time, and the tiles' sum is
    bit for bit the per-tile pass's."""
    sc = _scene(size, size, n_sub)
    sc.view = synth.perspective_view((0.5, 2.3, 0.9), (0.5, 0.5, 0.5), size, size)
    sc.m, sc.bias = 4, synth.default_bias(4)
    r = apc.Renderer(ctx, sc)
    want = []
    for k in range(n_sub):
        one = r.subs[k:k + 1]
        n = ctx.moments_pass_tiles(r.mesh, r.view, r.tf, 4, one, None, None, by_pair=True)
        tiles = torch.empty((n, 5, 64), device="cuda")
        bins = torch.empty(n, dtype=torch.int32, device="cuda")
        assert ctx.moments_pass_tiles(r.mesh, r.view, r.tf, 4, one, tiles, bins, by_pair=True) == n
        want.append(bins.long() * n_sub + k)
    want = torch.cat(want).sort().values
    tiles = torch.empty((len(want), 5, 64), device="cuda")
    bins = torch.empty(len(want), dtype=torch.int32, device="cuda")
    assert ctx.moments_pass_tiles(r.mesh, r.view, r.tf, 4, r.subs, tiles, bins, by_pair=True) == len(want)
    assert torch.equal(bins.long(), want)
    ctx.sum_moment_tiles(tiles, bins, len(want), n_sub, 4, size, size, r.moments)
    by_pair = r.moments.clone()
    try:
        ctx.set_dispatch(apc.APC_DISPATCH_QUEUE)
        ctx.moments_pass(r.mesh, r.view, r.tf, 4, r.subs, r.moments, global_sum=True)
        torch.cuda.synchronize()
    finally:
        ctx.set_dispatch(apc.APC_DISPATCH_GRID)
    assert torch.equal(by_pair, r.moments)
