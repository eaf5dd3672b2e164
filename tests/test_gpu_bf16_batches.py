"""BF16 MLP at the edges of its batches (64 samples gathered, 32 from staged
bricks): a sample's colour does not depend on the batch it is in, so a call's
rays equal the same rays of a longer call bit for bit, in either order."""
import pytest
import torch

import synth
from helpers import print_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hashed", [False, True])
@pytest.mark.parametrize("storage", [torch.float32, torch.float16])
@pytest.mark.parametrize("n", [1, 31, 33, 63, 64, 65, 8 * 64, 8 * 64 * 3 + 1, 2049])
def test_batch_edges(n, storage, hashed):
    import paper_2404_11852_amd as cic
    print_case("BF16 MLP, %d single-sample rays, %s, hashed %s" % (n, storage, hashed))
    dens, feats = synth.make_scene(24, seed=0)
    dens = dens * 0 + 50.0
    henc = synth.make_hash_tables(seed=3, res=(8, 16, 32, 64), log2_size=12) if hashed else None
    m = cic.Model(dens, feats, synth.make_mlp(1, bias_std=0.1), storage=storage, density_shift=0.0,
                  compute=cic.CIC_BF16, hash_enc=henc)
    o, d = (torch.from_numpy(t).cuda() for t in synth.random_rays(5000, seed=21, aim_half=1.2))
    whole = cic.render_rays(m, cic.make_opts(1), o, d)[0]
    assert float(whole[:n].std()) > 1e-3 or n == 1
    for order in (cic.CIC_ORDER_RAY, cic.CIC_ORDER_VOXEL):
        rgb = cic.render_rays(m, cic.make_opts(1, order=order), o[:n], d[:n])[0]
        assert torch.equal(rgb, whole[:n])
