"""Occupancy build at the edges of its tiles (8 voxels along x and 63 along z
per wavefront): bytes equal the oracle's on grids of ragged sizes."""
import numpy as np
import pytest
import torch

import oracle
import synth
from helpers import print_case, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("res", [(2, 2, 2), (9, 3, 64), (10, 2, 65), (8, 4, 63), (17, 5, 127), (18, 3, 128), (3, 40, 190)])
@pytest.mark.parametrize("storage", [torch.float32, torch.float16])
def test_occupancy_tiles(res, storage):
    import paper_2404_11852_amd as cic
    print_case("occupancy, %s grid, %s" % (res, storage))
    rng = np.random.default_rng(sum(res))
    # raw values on both sides of the threshold, mostly below it
    dens = np.where(rng.random(res) < 0.04, 9.0, -2.0).astype(np.float32) + rng.normal(0, 0.5, res).astype(np.float32)
    dens = dens.astype(np.float16).astype(np.float32)
    feats = np.zeros(res + (12,), np.float32)
    mlp = synth.make_mlp(1)
    m = cic.Model(dens, feats, mlp, storage=storage, density_shift=synth.DENSITY_SHIFT)
    got = to_np(m.build_occupancy(synth.OCC_SIGMA))
    want = oracle.build_occupancy(oracle.Model(dens, feats, mlp, density_shift=synth.DENSITY_SHIFT), synth.OCC_SIGMA)
    want = np.asarray(want).reshape(got.shape)
    assert np.array_equal(got, want)
    assert want.size < 9 or 0 < want.sum() < want.size
