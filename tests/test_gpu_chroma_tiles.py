"""4:2:0 handles through the tile kernel's staged chroma planes: equal to the
per-ray render bit for bit, at the smallest planes and across block sizes."""

import numpy as np
import pytest

import lfscene
import oracle
from conftest import crop_lf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block,h,w,levels", [(4, 8, 8, 2), (4, 24, 40, 3), (8, 16, 48, 2), (16, 64, 32, 1), (32, 64, 64, 2)])
def test_equal_to_per_ray(block, h, w, levels):
    import torch

    from paper_1902_09396_amd import lf

    cfg = lfscene.get_config("tiny", levels=levels, step=[4] * levels, win=[4] * levels, t_ref=[0] * levels,
                             t_pred=[0] * levels, block=block)
    cfg["enc"]["chroma420"] = True
    field = lf.LightField(oracle.encode(crop_lf("tiny", 7, 5, h, w), cfg["enc"]))
    for cams in (lfscene.random_pinhole_cameras(5, 7, 5, w, h, 45, 19, seed=block),
                 lfscene.camera_path_orbit(13, 7, 5, w, h, 45, 19, radius=1.5),
                 lfscene.projective_warp(lfscene.random_pinhole_cameras(3, 7, 5, w, h, 45, 19, seed=3), 2e-3, 1e-3)):
        dc = torch.from_numpy(np.ascontiguousarray(cams)).cuda()
        assert torch.equal(field.render_views(dc, 45, 19), field.render_views(dc, 45, 19, per_ray=True))
