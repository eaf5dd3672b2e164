"""Float32 MLP: the samples that float32 arithmetic computes again cost float32
arithmetic, not more.

Bound: the matrix cores do float32 products at a sixteenth of the float16 rate,
of which the split takes three, so a call whose every sample is computed again
may take the split's time and 16 / 3 of it."""
import numpy as np
import pytest
import torch

import helpers
import synth

pytestmark = pytest.mark.gpu


def _time(feats_scale, w0_scale):
    import paper_2404_11852_amd as cic
    dens, feats = synth.make_scene(24, seed=0)
    mlp = synth.make_mlp(1, bias_std=0.05)
    mlp["w0"][:, :12] *= np.float32(w0_scale)
    pair = helpers.Pair(24, dens=np.full_like(dens, 50.0), feats=feats * np.float32(feats_scale), mlp=mlp, shift=0.0)
    o, d = (torch.from_numpy(t).cuda() for t in synth.random_rays(200000, seed=2, aim_half=1.2))
    opts, best = cic.make_opts(8), 1e9
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        cic.render_rays(pair.gpu, opts, o, d)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


# feature columns far below the direction's; features beyond any float16; none a number
@pytest.mark.parametrize("feats,w0", [(1.0, 2.0 ** -18), (1e6, 1e-6), (1e30, 1e-30), (np.nan, 1.0)])
def test_cost(feats, w0):
    helpers.print_case("float32 MLP, every sample again, features x %g, W0's x %g" % (feats, w0))
    plain, got = _time(1.0, 1.0), _time(feats, w0)
    print("%.3f ms, %.3f ms" % (plain, got))
    assert got <= (1 + 16 / 3) * plain
