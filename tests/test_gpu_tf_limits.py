"""Extinctions beyond any cap: an infinite kappa, and one whose product with alpha overflows, make every piece with
some alpha as opaque as the cap allows, and leave pieces without alpha out, as the largest finite values do."""
import numpy as np
import pytest

import synth
from test_gpu_parity import apc, ctx  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [4, 8])
@pytest.mark.parametrize("kappa,scale", [(np.inf, 1.0), (3e38, 4.0)])
def test_infinite_extinction(apc, ctx, m, kappa, scale):
    sc = synth.scene_tiny()
    sc.view = synth.ortho_view_z(40, 40)
    sc.m, sc.bias = m, synth.default_bias(m)
    tf = synth.make_tf(12, n_entries=64)
    tf[:, 3] = np.where(np.arange(64) % 16 < 6, 0.0, np.maximum(tf[:, 3], 0.01)) * scale
    sc.tf = np.ascontiguousarray(tf)
    out = []
    for k in (1e30, kappa):
        sc.kappa = k
        r = apc.Renderer(ctx, sc)
        for kw in (dict(global_sum=True), dict(global_sum=True, resolve_by_pair=True),
                   dict(global_sum=True, keep=True), dict(global_sum=True, keep=True), dict()):
            r.frame(**kw)
            torch.cuda.synchronize()
            out.append((r.moments.clone(), r.rgba.clone()))
    assert float(out[0][0][0].max()) >= sc.absorbance_max
    for (a, b), (c, d) in zip(out[:5], out[5:]):
        assert torch.equal(a, c) and torch.equal(b, d)
