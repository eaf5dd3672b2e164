"""Float32 MLP on float32 products: whole calls (weights outside the split's
limits) and single samples (features beyond 2^60), dense grids and the
multi-level encoding, both orders, sample counts around the 16- and 32-sample
steps.  Tolerance: the renderer's 1e-5; both orders give the same bits."""
import numpy as np
import pytest
import torch

import oracle
import synth
from helpers import TOL, print_case, to_np

pytestmark = pytest.mark.gpu

HASH = dict(res=(24, 48, 96, 192), log2_size=12)


@pytest.mark.parametrize("n", [1, 16, 17, 33, 256 * 33 + 5])
@pytest.mark.parametrize("what,hashed,storage", [
    ("weights", False, torch.float32), ("weights", False, torch.float16), ("weights", True, torch.float32),
    ("weights", True, torch.float16), ("samples", False, torch.float32), ("samples", True, torch.float32)])
def test_float32_products(n, what, hashed, storage):
    import paper_2404_11852_amd as cic
    print_case("float32 products for %s, hashed %d, %s, %d samples" % (what, hashed, storage, n))
    dens, feats = synth.make_scene(24, seed=0)
    dens = np.full_like(dens, 50.0)
    enc = synth.make_hash_tables(31, **HASH) if hashed else None
    mlp = synth.make_mlp(1, bias_std=0.05)
    if what == "weights":
        mlp["w1"][::2] *= np.float32(2.0 ** -30)
        mlp["b1"][::2] *= np.float32(2.0 ** -30)
        mlp["w2"][:, ::2] *= np.float32(2.0 ** 30)
    else:   # about half of the samples: the entries of one feature, where positive
        big = np.float32(1e25)
        mlp["w0"][:, 4] /= big
        if hashed:
            t = enc["tables"].copy()
            t[1, ..., 1] = np.where(t[1, ..., 1] > 0, t[1, ..., 1] * big, 0)
            enc = dict(enc, tables=t)
        else:
            feats[..., 4] = np.where(feats[..., 4] > 0, feats[..., 4] * big, 0)
    gpu = cic.Model(dens, None if hashed else feats, mlp, storage=storage, density_shift=0.0, hash_enc=enc)
    if storage == torch.float16:
        dens, feats = (t.astype(np.float16).astype(np.float32) for t in (dens, feats))
        enc = enc and dict(enc, tables=enc["tables"].astype(np.float16).astype(np.float32))
    orc = oracle.Model(dens, None if hashed else feats, mlp, density_shift=0.0, hash_enc=enc)
    o, d = (np.ascontiguousarray(t[-n:]) for t in synth.random_rays(n + 40, seed=21, aim_half=1.2))
    want, _, _ = oracle.render_rays(orc, oracle.opts(1, 0.0), o, d)
    got = [to_np(cic.render_rays(gpu, cic.make_opts(1, order=k), torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda())[0])
           for k in (cic.CIC_ORDER_RAY, cic.CIC_ORDER_VOXEL)]
    print("max error %.2e" % np.abs(got[0] - want).max())
    assert np.all((want > 0.05) & (want < 0.95))   # (no saturated colours)
    assert np.abs(got[0] - want).max() <= TOL
    assert np.array_equal(got[0], got[1])
