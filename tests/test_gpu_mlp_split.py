"""Float32 MLP on split float16 products: batch edges, the range of the split
and what happens beyond it, against the float64 oracle.

Tolerance: the layer is as exact as float32 arithmetic, so the renderer's
1e-5 on colours holds; scaling the hidden layers by s and the output weights
by 1/s changes no relative error, so it holds at every scale."""
import numpy as np
import pytest
import torch

import helpers
import oracle
import synth

pytestmark = pytest.mark.gpu


def _one_sample_pair(scale_feat=1.0, scale_w0=1.0, w2=1.0, occupancy=False):
    dens, feats = synth.make_scene(24, seed=0)
    mlp = synth.make_mlp(1, bias_std=0.05)
    mlp["w0"], mlp["b0"] = mlp["w0"] * np.float32(scale_w0), mlp["b0"] * np.float32(scale_w0)
    mlp["b1"] = mlp["b1"] * np.float32(1.0 / w2)
    mlp["w2"] = mlp["w2"] * np.float32(w2)
    return helpers.Pair(24, dens=np.full_like(dens, 50.0), feats=feats * np.float32(scale_feat), mlp=mlp, shift=0.0)


def _rays(n):
    o, d = synth.random_rays(n + 40, seed=21, aim_half=1.2)
    return np.ascontiguousarray(o[-n:]), np.ascontiguousarray(d[-n:])


def _render(model, order, o, d):
    import paper_2404_11852_amd as cic
    opts = cic.make_opts(1, order=cic.CIC_ORDER_VOXEL if order else cic.CIC_ORDER_RAY)
    rgb, _, _ = cic.render_rays(model, opts, torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda())
    return helpers.to_np(rgb)


@pytest.mark.parametrize("n", [1, 31, 32, 33, 255, 257, 8 * 32, 8 * 32 * 3 + 1, 2049])
def test_batch_edges(n):
    helpers.print_case("split MLP, %d single-sample rays" % n)
    pair = _one_sample_pair()
    o, d = _rays(n)
    want, _, _ = oracle.render_rays(pair.orc, oracle.opts(1, 0.0), o, d)
    got = _render(pair.gpu, 0, o, d)
    helpers.compare(got, want)
    assert np.array_equal(got, _render(pair.gpu, 1, o, d))


# features beyond 65504 and activations beyond it are computed again in float32
@pytest.mark.parametrize("scale_feat,scale_w0,w2", [(1e-4, 1.0, 1.0), (1.0, 1e-6, 1e6), (1.0, 1e6, 1e-6),
                                                    (3e3, 1.0, 1.0 / 3e3), (2e4, 1.0, 5e-5), (1e8, 1.0, 1e-8),
                                                    (1e25, 1.0, 1e-25)])
def test_scales(scale_feat, scale_w0, w2):
    helpers.print_case("split MLP, features x %g, W0 x %g" % (scale_feat, scale_w0))
    pair = _one_sample_pair(scale_feat, scale_w0, w2)
    o, d = _rays(1500)
    want, _, _ = oracle.render_rays(pair.orc, oracle.opts(1, 0.0), o, d)
    got = _render(pair.gpu, 0, o, d)
    helpers.compare(got, want)
    assert np.array_equal(got, _render(pair.gpu, 1, o, d))


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf, 3e38])
def test_poisoned_vertex(value):
    """Samples that touch a vertex with a value float32 arithmetic makes
    non-finite (or that leaves the split's range) do not change the others'."""
    helpers.print_case("split MLP, one vertex %g" % value)
    pair = _one_sample_pair()
    o, d = _rays(3000)
    clean = _render(pair.gpu, 0, o, d)
    feats = pair.feats.copy()
    feats[12, 12, 12, 5] = value
    pair2 = helpers.Pair(24, dens=pair.dens, feats=feats, mlp=pair.mlp, shift=0.0)
    got = _render(pair2.gpu, 0, o, d)
    # which rays' sample lies in the vertex's eight cells
    marks = np.zeros_like(pair.feats)
    marks[12, 12, 12, 5] = 1e3
    touched = (_render(helpers.Pair(24, dens=pair.dens, feats=pair.feats + marks, mlp=pair.mlp, shift=0.0).gpu, 0, o, d)
               != clean).any(axis=1)
    assert 0 < touched.sum() < 3000
    assert np.array_equal(got[~touched], clean[~touched])
    if np.isnan(value):
        # (the interpolation gives a NaN either sign, and the integer ReLU
        # keeps the positive ones)
        assert np.isnan(got[touched]).any()
    ok = np.isnan(got) | ((got >= 0) & (got <= 1))
    assert ok.all()
