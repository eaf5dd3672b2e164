"""Voxel-order bucketing at the edges of its rule for rays per block (per-run
counters below 2048 rays, then blocks of 16 to 256 rays, the last one ragged):
voxel order must give ray order's bits, which it does only if every sample's
place in the permutation is taken exactly once."""
import pytest
import torch

import synth
from helpers import print_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("res,n_rays", [(33, 2047), (33, 2048), (33, 2049), (33, 16 * 512 - 1), (33, 32 * 512),
                                        (33, 64 * 512 + 1), (33, 128 * 512 + 100), (201, 2100), (209, 2100)])
def test_voxel_order_equals_ray_order(res, n_rays):
    import paper_2404_11852_amd as cic
    print_case("bucketing, %d^3 grid, %d rays" % (res, n_rays))   # 201: 15,625 bricks, 209: 17,576 (no LDS histogram)
    dens = torch.full((res,) * 3, 1.0)
    feats = torch.randn((res,) * 3 + (12,), generator=torch.Generator().manual_seed(n_rays)) if res < 100 else \
        torch.linspace(-1.0, 1.0, 12).expand((res,) * 3 + (12,))
    m = cic.Model(dens, feats, synth.make_mlp(1, bias_std=0.1), density_shift=0.0)
    o, d = (torch.from_numpy(t).cuda() for t in synth.random_rays(n_rays, seed=3))
    got = []
    for order in (cic.CIC_ORDER_RAY, cic.CIC_ORDER_VOXEL):
        n = torch.zeros(1, dtype=torch.int64, device="cuda")
        got.append((*cic.render_rays(m, cic.make_opts(40, order=order), o, d, n_eval=n), n))
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("n_rays", [1, 3, 1023, 1025, 4096, 4097, 16381, 16385, 2048 * 9 + 1])
def test_scan_edges(n_rays):
    """Record offsets at the edges of the one-block scan and of the blocks of
    the longer one: rays rendered together equal rays rendered in two calls."""
    import paper_2404_11852_amd as cic
    print_case("scan, %d rays" % n_rays)
    dens, feats = synth.make_scene(24, seed=0)
    m = cic.Model(dens, feats, synth.make_mlp(1, bias_std=0.1), density_shift=synth.DENSITY_SHIFT)
    m.build_occupancy(synth.OCC_SIGMA)
    o, d = (torch.from_numpy(t).cuda() for t in synth.random_rays(n_rays, seed=4))
    opts = cic.make_opts(33, 1e-4, True)
    whole = cic.render_rays(m, opts, o, d)
    k = n_rays // 3
    parts = [cic.render_rays(m, opts, o[a:b], d[a:b]) for a, b in ((0, k), (k, n_rays)) if b > a]
    for i, t in enumerate(whole):
        assert torch.equal(t, torch.cat([p[i] for p in parts]))


@pytest.mark.parametrize("n_rays,samples", [(32767, 130), (32769, 63), (32771, 200), (262143, 65), (262145, 129),
                                            (262151, 64)])
def test_compaction_edges(n_rays, samples):
    """Records of 1, 4 or 8 rays per wavefront with ragged last groups, rays of
    up to three chunks of 64 samples: rays rendered together equal rays
    rendered in small calls."""
    import paper_2404_11852_amd as cic
    print_case("compaction, %d rays, %d samples" % (n_rays, samples))
    dens, feats = synth.make_scene(24, seed=0)
    m = cic.Model(dens, feats, synth.make_mlp(1, bias_std=0.1), density_shift=synth.DENSITY_SHIFT)
    if samples < 100:
        m.build_occupancy(synth.OCC_SIGMA)
    o, d = (torch.from_numpy(t).cuda() for t in synth.random_rays(n_rays, seed=4))
    opts = cic.make_opts(samples, 0.0, samples < 100)
    whole = cic.render_rays(m, opts, o, d)
    parts = [cic.render_rays(m, opts, o[a:a + 30000], d[a:a + 30000]) for a in range(0, n_rays, 30000)]
    for i, t in enumerate(whole):
        assert torch.equal(t, torch.cat([p[i] for p in parts]))
