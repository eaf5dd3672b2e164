"""March of whole frames: the form that the rule chooses for a frame is not
slower than the march of the same rays given one by one.

Bound: 8% over the smallest of several alternating runs, which is more than
they differ by."""
import pytest
import torch

import synth
from helpers import print_case

pytestmark = pytest.mark.gpu


def _march_ms(call):
    from paper_2404_11852_amd import _lib
    _lib.timing_enable(True)
    call()
    torch.cuda.synchronize()
    t = _lib.timing_read()
    _lib.timing_enable(False)
    return [v[0] for k, v in t.items() if "march" in str(k).lower()][0]


@pytest.mark.parametrize("res,occ", [(64, True), (96, True), (96, False)])
@pytest.mark.parametrize("width,height", [(450, 450), (512, 512), (640, 480), (800, 800)])
def test_not_slower(res, occ, width, height):
    print_case("march rule, %dx%d, grid %d, occupancy %d" % (width, height, res, occ))
    import paper_2404_11852_amd as cic
    dens, feats = synth.make_scene(res, seed=0)
    model = cic.Model(dens, feats, synth.make_mlp(1), storage=torch.float16, density_shift=synth.DENSITY_SHIFT)
    if occ:
        model.build_occupancy(synth.OCC_SIGMA)
    opts = cic.make_opts(256, use_occupancy=occ)
    f, cx, cy = synth.intrinsics(width, height)
    cam = cic.make_camera(width, height, f, cx, cy, synth.as_f32(synth.orbit_pose(1)))
    o, d = cic.generate_rays(cam)
    frame = rays = 1e9
    for _ in range(9):
        frame = min(frame, _march_ms(lambda: cic.render_frame(model, opts, cam)))
        rays = min(rays, _march_ms(lambda: cic.render_rays(model, opts, o, d)))
    print("frame %.3f ms, rays %.3f ms" % (frame, rays))
    assert frame <= 1.08 * rays
