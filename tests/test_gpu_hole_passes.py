"""SpaRW targets from no hole to nothing but holes: the hole pass strides over
the rays the device counted, and its pixels are those of a full render."""
import pytest
import torch

import synth
from helpers import print_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size,compute", [((64, 48), "f32"), ((201, 173), "f32"), ((640, 450), "f32"), ((640, 450), "bf16")])
@pytest.mark.parametrize("motion", ["none", "shift", "turn"])
def test_holes_equal_full_render(size, compute, motion):
    import paper_2404_11852_amd as cic
    W, H = size
    print_case("hole pass, %dx%d %s, %s" % (W, H, compute, motion))
    dens, feats = synth.make_scene(32, seed=0)
    m = cic.Model(dens, feats, synth.make_mlp(1, bias_std=0.1), density_shift=synth.DENSITY_SHIFT,
                  compute=cic.CIC_BF16 if compute == "bf16" else cic.CIC_F32)
    m.build_occupancy(synth.OCC_SIGMA)
    f, cx, cy = synth.intrinsics(W, H)
    pose = synth.as_f32(synth.orbit_pose(0))
    cam = cic.make_camera(W, H, f, cx, cy, pose)
    opts = cic.make_opts(40, 1e-4, True)
    rgb, dz, _ = cic.render_frame(m, opts, cam)
    T = torch.eye(4)[:3].clone()
    if motion == "shift":
        T[0, 3] = 0.05
    elif motion == "turn":   # the reference lies behind the target camera
        T[0, 0] = T[2, 2] = -1.0
    out, oz, mask, nm = cic.render_frame_sparw(m, opts, cam, rgb, dz, cam, T.reshape(-1).numpy())
    holes = mask.bool()
    assert int(nm) == int(holes.sum())
    print("%d holes of %d" % (int(nm), W * H))
    assert motion == "none" or int(nm) > 0
    # a hole's pixel is rendered from its own ray, as in the full frame (the BF16 batches differ in nothing else)
    assert torch.equal(out[holes], rgb[holes])
    assert torch.equal(oz[holes], dz[holes])
