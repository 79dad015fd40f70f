"""The walk, the chord queue of stage one and the chord ring of stage two where they can go wrong, against the
FP64 oracle with the bars of tests/test_gpu_parity.py: rays exactly through vertices and edges (zero side
products), chords of one piece and of hundreds (a queue that never fills, one that always is full), more
boundary faces in a bin than one stage holds (32) and more entries than one round holds (8), and the smallest
and largest transfer-function tables."""
import math

import numpy as np
import pytest

import oracle
import synth
from test_gpu_parity import _check_moments, _flat_moments, _np, _render, apc, ctx  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _check_frame(apc, ctx, sc, ref):
    """Moments, image, pieces and the agreement of the two walks of one frame with the oracle's."""
    r, rgba = _render(apc, ctx, sc)
    W, H = sc.view["width"], sc.view["height"]
    _check_moments(sc, np.arange(W * H), _flat_moments(r.moments), ref)
    d = _np(rgba).reshape(-1, 4) - ref["rgba"]
    assert np.abs(d).max() <= 2e-3 and math.sqrt(np.mean(d ** 2)) <= 5e-4
    ctx.counters(reset=True)
    ctx.moments_pass(r.mesh, r.view, r.tf, sc.m, r.subs, r.moments, None, global_sum=True)
    torch.cuda.synchronize()
    one = ctx.counters(reset=True)
    ctx.resolve_pass(r.mesh, r.view, r.tf, r.mboit, r.moments, r.subs, r.rgba, finalize=True)
    torch.cuda.synchronize()
    two = ctx.counters()
    assert one["walk_step_limit"] == 0
    for k in ("pieces", "tet_steps", "entries", "segments"):
        assert two[k] == one[k], (k, one[k], two[k])
    assert abs(one["pieces"] - ref["n_pieces"]) <= 1e-4 * ref["n_pieces"] + 2
    return one


def _with_order(sc, m):
    sc.m, sc.bias = m, synth.default_bias(m)
    return sc


@pytest.mark.parametrize("m", [4, 8])
def test_rays_through_vertices_and_edges(apc, ctx, m):
    """A grid without jitter seen along z with every pixel centre on a grid line or a cell's diagonal: each
    ray runs along edges and through vertices, so most side products are exact zeros, decided by vertex ids.
    The walk gives each ray every point of the cube once.  The oracle clips each tet by itself and counts a
    ray inside a shared face or edge with every tet around it, so its camera stands 1e-6 of a cell aside: the
    field is continuous, and its rays then meet no vertex or edge."""
    n = 8
    mesh = synth.grid_mesh(n, 4, 3, n_gauss=4, jagged_seed=11, jitter=0.0)
    W = 2 * n - 1  # centres at 1/16, 2/16, ... 15/16: inside, on planes and cell centres
    right, down = np.array([1.0 / (2 * n), 0, 0]), np.array([0, 1.0 / (2 * n), 0])
    eye = np.array([0.0, 0.0, -1.0]) + 0.5 * (right + down)
    view = dict(width=W, height=W, projection=0, eye=tuple(eye), dir=(0.0, 0.0, 1.0), right=tuple(right),
                down=tuple(down))
    sc = _with_order(synth.Scene(name="ties", mesh=mesh, tf=synth.make_tf(3), s_min=float(mesh.scalar.min()),
                                 s_max=float(mesh.scalar.max()), kappa=4.0, absorbance_max=10.0, view=view,
                                 step=0.03, m=m, alpha=5e-5, bias=synth.default_bias(m), eta=0.3), m)
    r, rgba = _render(apc, ctx, sc)
    aside = dict(view, eye=tuple(eye + np.array([1.0, 0.37, 0.0]) * 1e-6 / n))
    ref = oracle.render(synth.Scene(**{**sc.__dict__, "view": aside}))
    got = _flat_moments(r.moments)
    assert ref["moments"][0].min() > 0
    assert np.abs(got - ref["moments"]).max() <= 1e-5 * ref["moments"][0].max()
    d = _np(rgba).reshape(-1, 4) - ref["rgba"]
    assert np.abs(d).max() <= 2e-3 and math.sqrt(np.mean(d ** 2)) <= 5e-4
    assert ctx.counters()["walk_step_limit"] == 0


@pytest.mark.parametrize("m", [4, 6, 8])
@pytest.mark.parametrize("per_cell", [0.01, 1.0, 200.0])
def test_chords_of_one_piece_and_of_hundreds(apc, ctx, m, per_cell):
    """Steps of 100 cells (every chord one piece, no lattice point in the mesh), of one and of 1/200 cell."""
    sc = _with_order(synth.scene_tiny(), m)
    sc.view = synth.perspective_view(synth.sphere_eye(5), (0.5, 0.5, 0.5), 29, 21)
    sc.step = 1.0 / 16 / per_cell
    c = _check_frame(apc, ctx, sc, oracle.render(sc))
    if per_cell < 0.1:
        assert c["pieces"] <= 1.02 * c["tet_steps"]
    elif per_cell > 100:
        assert c["pieces"] >= 50 * c["tet_steps"]


@pytest.mark.parametrize("slabs,size", [(8, 24), (9, 24), (20, 13)])
def test_entries_and_faces_beyond_one_round(apc, ctx, slabs, size):
    """Interleaved slabs: each ray enters each subdomain `slabs` times (8 entries are held at once), and at
    these image sizes a tile meets hundreds of boundary faces of each subdomain (32 are staged at once)."""
    sc = _with_order(synth.scene_slabs(n_ranks=2, slabs_per_rank=slabs, cells_per_slab=1, size=size), 8)
    ref = oracle.render(sc)
    c = _check_frame(apc, ctx, sc, ref)
    assert c["entries"] >= 2 * slabs * size * size
    assert (c["entry_overflow"] > 0) == (slabs > 8)


@pytest.mark.parametrize("entries", [2, 3, 1024])
@pytest.mark.parametrize("m", [4, 8])
def test_smallest_and_largest_tables(apc, ctx, entries, m):
    """Transfer functions of 2, 3 and 1024 entries over half of the scalar range (the rest clamps to the ends)."""
    sc = _with_order(synth.scene_tiny(), m)
    sc.view = synth.ortho_view_z(40, 40)
    sc.tf = np.ascontiguousarray(synth.make_tf(12, n_entries=1024)[np.linspace(0, 1023, entries).astype(int)])
    lo, hi = sc.s_min, sc.s_max
    sc.s_min, sc.s_max = lo + 0.25 * (hi - lo), lo + 0.75 * (hi - lo)
    _check_frame(apc, ctx, sc, oracle.render(sc))


@pytest.mark.parametrize("m", [4, 6, 8])
@pytest.mark.parametrize("per_cell", [0.01, 0.5, 12.0])
def test_kept_pieces_of_uneven_rays(apc, ctx, m, per_cell):
    """Kept pieces evaluated a lane per pixel: rays of no piece, of a few (less than a batch of 4, a group of 8
    or a chunk of 64) and of many chunks side by side in a tile, against the oracle and the plain form (whose
    colour sums are FP32 throughout: the bar of the other forms, 2e-5)."""
    sc = _with_order(synth.scene_tiny(), m)
    sc.view = synth.perspective_view(synth.sphere_eye(5), (0.5, 0.5, 0.5), 61, 43)
    sc.step = 1.0 / 16 / per_cell
    ref = oracle.render(sc)
    r = apc.Renderer(ctx, sc)
    for _ in range(3):  # the first frames size the piece pool
        r.rgba.fill_(-1.0)
        r.frame(global_sum=True, keep=True)
    torch.cuda.synchronize()
    assert ctx.timings()["eval_ms"] > 0
    kept = r.rgba.clone()
    d = _np(kept).reshape(-1, 4) - ref["rgba"]
    assert np.abs(d).max() <= 2e-3 and math.sqrt(np.mean(d ** 2)) <= 5e-4
    r.frame(global_sum=True)
    torch.cuda.synchronize()
    assert float((r.rgba - kept).abs().max()) <= 2e-5
