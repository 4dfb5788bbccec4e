"""Calls of one view, and batches of unrelated views, whose groups take the
plan without lookups: equal to the per-ray render bit for bit."""

import numpy as np
import pytest

import lfscene
import oracle
from conftest import crop_lf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("na,nb,levels,block", [(1, 1, 1, 16), (7, 1, 3, 8), (2, 8, 1, 16), (8, 8, 2, 4), (8, 7, 8, 16), (8, 8, 4, 16)])
def test_equal_to_per_ray(na, nb, levels, block):
    import torch

    from paper_1902_09396_amd import lf

    cfg = lfscene.get_config("tiny", levels=levels, step=[4] * levels, win=[4] * levels, t_ref=[0] * levels,
                             t_pred=[0] * levels, block=block)
    field = lf.LightField(oracle.encode(crop_lf("tiny", na, nb, 64, 48), cfg["enc"]))
    near = lfscene.random_pinhole_cameras(6, na, nb, 48, 64, 70, 33, seed=na)
    # eyes far from the view plane: tiles that reach many views, up to beyond the budgets
    wide = lfscene.random_pinhole_cameras(6, na, nb, 48, 64, 70, 33, seed=nb, ez_range=(-4.0, -1.0), rho=0.3)
    for cams in (near, wide, np.concatenate([near, wide])[[0, 6, 6, 1, 1, 7]]):
        dc = torch.from_numpy(np.ascontiguousarray(cams)).cuda()
        ref = field.render_views(dc, 70, 33, per_ray=True)
        assert torch.equal(field.render_views(dc, 70, 33), ref)
        for v in range(len(cams)):
            assert torch.equal(field.render_views(dc[v:v + 1], 70, 33), ref[v:v + 1])
