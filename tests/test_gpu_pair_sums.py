"""The ordered FP64 sum of (tile, subdomain) pairs into the moment image, on made-up pairs: bit for bit the sum
that numpy takes in the same order, at sizes where the search for a tile's pairs and the tiles at the image's
edges can go wrong."""
import numpy as np
import pytest

from test_gpu_parity import apc, ctx  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H,n_sub,m,tw,density", [
    (1, 1, 1, 4, 8, 1.0), (1, 1, 200, 8, 8, 1.0),      # one tile; more pairs than a wavefront's lanes
    (64, 64, 64, 6, 8, 1.0), (65, 63, 65, 4, 16, 0.5),  # a tile's pairs fill the lanes exactly, and not quite
    (200, 120, 3, 8, 8, 0.3), (33, 70, 128, 6, 1, 0.9), (70, 5, 7, 4, 64, 0.02),
    (40, 40, 5, 8, 8, 0.0),                             # no pair at all
])
def test_pair_sum_is_the_ordered_sum(apc, ctx, W, H, n_sub, m, tw, density):
    rng = np.random.default_rng(W * 7 + H + n_sub)
    th, m1 = 64 // tw, m + 1
    tx, ty = -(-W // tw), -(-H // th)
    bins = np.flatnonzero(rng.random(tx * ty * n_sub) < density).astype(np.int32)
    tiles = rng.uniform(-3.0, 3.0, (len(bins), m1, 64)).astype(np.float32)
    want = np.zeros((m1, ty * th, tx * tw))
    for p, b in enumerate(bins):  # ascending: the pairs of a tile in slot order
        t = b // n_sub
        y, x = t // tx * th, t % tx * tw
        want[:, y:y + th, x:x + tw] += tiles[p].astype(np.float64).reshape(m1, th, tw)
    want = want[:, :H, :W].astype(np.float32)
    before = ctx.tile_shape()[0]
    ctx.set_tile_shape(tw)
    try:
        out = torch.full((m1, H, W), -1.0, device="cuda")
        ctx.sum_moment_tiles(torch.from_numpy(tiles).cuda(), torch.from_numpy(bins).cuda(), len(bins), n_sub, m, H, W,
                             out)
        torch.cuda.synchronize()
    finally:
        ctx.set_tile_shape(before)
    assert np.array_equal(out.cpu().numpy(), want)
