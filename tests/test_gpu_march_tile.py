"""March of whole frames in 8 x 8 pixel tiles (196,608 pixels and more): the
same samples, weights, transmittances and depths as the march of single rays,
bit for bit, so a frame equals its pixels rendered as rays; sizes that are no
multiple of 8, sample counts that are no multiple of 16 or 64, with and
without skipping and termination, both grid types, passes that cut rows."""
import pytest
import torch

import synth
from helpers import cams, print_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,res,n,occ,et,storage", [
    (512, 384, 48, 64, True, 1e-4, torch.float32), (601, 331, 65, 100, True, 1e-4, torch.float16),
    (449, 449, 48, 129, False, 0.0, torch.float32), (803, 250, 33, 17, False, 1e-3, torch.float16),
    (1999, 99, 48, 15, True, 0.0, torch.float32), (455, 433, 96, 256, True, 0.5, torch.float32),
    (520, 380, 24, 1, False, 1e-4, torch.float32), (450, 440, 40, 1024, True, 1e-4, torch.float16)])
def test_tiles_equal_rays(w, h, res, n, occ, et, storage):
    import paper_2404_11852_amd as cic
    print_case("tile march %dx%d, %d^3, %d samples, occ %s, et %g, %s" % (w, h, res, n, occ, et, storage))
    assert w * h >= 196608
    dens, feats = synth.make_scene(res, seed=1)
    m = cic.Model(dens, feats, synth.make_mlp(1, bias_std=0.1), storage=storage, density_shift=synth.DENSITY_SHIFT)
    if occ:
        m.build_occupancy(synth.OCC_SIGMA)
    cam, _ = cams(w, h, synth.orbit_pose(20))
    opts = cic.make_opts(n, et, occ)
    k = torch.zeros(2, dtype=torch.int64, device="cuda")
    rgb, dz, acc = cic.render_frame(m, opts, cam, n_eval=k[:1])
    o, d = cic.generate_rays(cam)
    rgb2, dt2, acc2 = cic.render_rays(m, opts, o, d, n_eval=k[1:])
    assert int(k[0]) == int(k[1]) > 0
    assert torch.equal(rgb, rgb2) and torch.equal(acc, acc2)
    fwd = torch.tensor([cam.c2w[2], cam.c2w[6], cam.c2w[10]], device="cuda")
    seen = acc >= opts.void_acc
    want = dt2[seen].double() / acc[seen].double() * (d[seen].double() * fwd.double()).sum(1)
    assert torch.all(torch.isinf(dz[~seen])) and torch.allclose(dz[seen].double(), want, rtol=1e-5, atol=0)
    # two passes, the first cutting a row: the march of single rays
    try:
        from paper_2404_11852_amd import _lib
        cic.set_workspace_limit(_lib.workspace_bytes(_lib.OP_RENDER_FRAME, w * h - w // 2, m.grid, opts))
        part = cic.render_frame(m, opts, cam)
    finally:
        cic.set_workspace_limit(None)
    for a, b in zip(part, (rgb, dz, acc)):
        assert torch.equal(a, b)
