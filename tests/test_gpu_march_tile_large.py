"""The tile march at sizes above the lines from which whole frames take it
(250,000 pixels, with an occupancy grid 300,000): same bits as single rays."""
import pytest
import torch

from test_gpu_march_tile import test_tiles_equal_rays as _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,res,n,occ,et,storage", [
    (640, 480, 48, 64, True, 1e-4, torch.float32), (701, 431, 65, 100, True, 1e-4, torch.float16),
    (501, 501, 48, 129, False, 0.0, torch.float32), (1003, 250, 33, 17, False, 1e-3, torch.float16),
    (2999, 101, 48, 15, True, 0.0, torch.float32), (605, 501, 96, 256, True, 0.5, torch.float32),
    (520, 490, 24, 1, False, 1e-4, torch.float32), (600, 510, 40, 1024, True, 1e-4, torch.float16)])
def test_tiles_equal_rays_above_the_line(w, h, res, n, occ, et, storage):
    assert w * h >= (300000 if occ else 250000)
    _check(w, h, res, n, occ, et, storage)
