"""MLP adjoint on split float16 products: batch edges, the range of the split
and the float32 kernel beyond it, against the float64 oracle.

Tolerance: the adjoint's 1e-4 per tensor.  The scalings are powers of two that
leave the rendered function as it is, so they change no relative error."""
import numpy as np
import pytest
import torch

import oracle
import synth
from helpers import Pair, print_case, to_np

pytestmark = pytest.mark.gpu

NAMES = ("density", "features", "w0", "b0", "w1", "b1", "w2", "b2")


def _pair(feat=1.0, h1=1.0, h2=1.0):
    """Features x feat, first activations x h1, second ones x h2, the same outputs."""
    dens, feats = synth.make_scene(24, seed=4)
    mlp = synth.make_mlp(5, bias_std=0.1)
    f32 = np.float32
    mlp["w0"][:, :12] /= f32(feat)
    mlp["w0"], mlp["b0"] = mlp["w0"] * f32(h1), mlp["b0"] * f32(h1)
    mlp["w1"], mlp["b1"] = mlp["w1"] * f32(h2) / f32(h1), mlp["b1"] * f32(h2)
    mlp["w2"] = mlp["w2"] / f32(h2)
    return Pair(0, dens=dens, feats=feats * f32(feat), mlp=mlp)


def _backward(p, n_samples, o, d, d_rgb):
    import paper_2404_11852_amd as cic
    g = cic.render_backward(p.gpu, cic.make_opts(n_samples), *(torch.from_numpy(t).cuda() for t in (o, d, d_rgb)))
    torch.cuda.synchronize()
    return {k: to_np(v).astype(np.float64) for k, v in g.items()}


def _check(p, n_samples, o, d, d_rgb):
    g = _backward(p, n_samples, o, d, d_rgb)
    og, _ = oracle.render_backward(p.orc, oracle.opts(n_samples, 0.0), o, d, d_rgb.astype(np.float64))
    for k in NAMES:
        r = np.linalg.norm(g[k] - og[k]) / max(np.linalg.norm(og[k]), 1e-300)
        print("%s rel %.2e" % (k, r))
        assert r <= 1e-4, (k, r)


def _case(n, seed=9):
    o, d = synth.random_rays(n, seed=seed)
    return o, d, np.random.default_rng(n).normal(0, 1e-3, (n, 3)).astype(np.float32)


@pytest.mark.parametrize("n,samples", [(1, 3), (2, 8), (5, 3), (17, 1), (127, 1), (33, 64), (300, 33)])
def test_batch_edges(n, samples):
    print_case("split adjoint, %d rays, %d samples" % (n, samples))
    _check(_pair(), samples, *_case(n))


# (2^110: beyond the split's range, the float32 kernel)
@pytest.mark.parametrize("feat,h1,h2,grad", [(-8, 0, 0, 0), (14, 0, 0, 0), (0, -10, 0, 0), (0, 14, 0, 0), (0, 0, -20, 0),
                                             (0, 0, 14, 0), (0, 0, 40, 0), (0, 0, 0, -50), (0, 0, 0, 60), (0, 0, 0, 118),
                                             (-30, 0, 0, 0), (30, 0, 0, 0), (110, 0, 0, 0), (0, -60, 0, 0), (0, 110, 0, 0)])
def test_scales(feat, h1, h2, grad):
    print_case("split adjoint, features 2^%d, h1 2^%d, h2 2^%d, gradient 2^%d" % (feat, h1, h2, grad))
    o, d, d_rgb = _case(400)
    _check(_pair(2.0 ** feat, 2.0 ** h1, 2.0 ** h2), 40, o, d, d_rgb * np.float32(2.0 ** grad))


@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_poisoned_gradient(value):
    """One ray's upstream gradient not finite: only vertices it reaches and the
    MLP's gradients follow it."""
    print_case("split adjoint, one gradient %g" % value)
    p = _pair()
    o, d, d_rgb = _case(600)
    clean = _backward(p, 40, o, d, d_rgb)
    poisoned = d_rgb.copy()
    poisoned[5] = value
    # the vertices of that ray's samples
    hit = ~np.isfinite(_backward(p, 40, o[5:6], d[5:6], poisoned[5:6])["features"]).all(axis=-1)
    assert hit.any() and not hit.all()
    got = _backward(p, 40, o, d, poisoned)
    assert np.array_equal(~np.isfinite(got["features"]).all(axis=-1), hit)
    a, b = got["features"][~hit], clean["features"][~hit]
    assert np.linalg.norm(a - b) <= 1e-4 * np.linalg.norm(b)
    assert not np.isfinite(got["w1"]).all()


@pytest.mark.parametrize("seed", range(6))
def test_scale_edges(seed):
    """Gradients and output weights with mantissas near 2, all of one sign, so
    that dp1 comes close to its bound."""
    print_case("split adjoint, dp1 at its bound, seed %d" % seed)
    p = _pair()
    rng = np.random.default_rng(seed)
    mlp = dict(p.mlp)
    mlp["w2"] = np.full_like(mlp["w2"], (1.25, 1.5, 1.75, 1.9, 1.99, 1.0)[seed] * 2.0 ** -4)
    mlp["b2"] = np.full_like(mlp["b2"], -0.5 * mlp["w2"][0, 0] * 128 * 0.3)
    q = Pair(0, dens=p.dens, feats=p.feats, mlp=mlp)
    o, d = synth.random_rays(500, seed=seed)
    d_rgb = np.repeat(rng.uniform(1.0, 2.0, (500, 1)).astype(np.float32), 3, axis=1) * np.float32(1e-3)
    _check(q, 24, o, d, d_rgb)


@pytest.mark.parametrize("n,dims", [(600, (18, 10, 26)), (2500, (9, 9, 9)), (40, (70, 66, 74))])
def test_segments(n, dims):
    """Feature gradients of bricks with 0 to over 512 samples (several segments)
    and of 1 to over 512 bricks (one or two levels of the segment's search)."""
    print_case("feature gradients, %d rays, grid %dx%dx%d" % (n, *dims))
    dens, feats = synth.make_scene(80, seed=2)
    a, b, c = dims
    p = Pair(0, dens=np.ascontiguousarray(dens[:a, :b, :c]), feats=np.ascontiguousarray(feats[:a, :b, :c]),
             mlp=synth.make_mlp(3, bias_std=0.1))
    _check(p, 50, *_case(n))
