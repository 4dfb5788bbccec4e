"""Block-sparse handles through the tile kernel: equal to their per-ray
render and to the dense handle bit for bit, every level."""

import numpy as np
import pytest

import lfscene
import oracle
from conftest import crop_lf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block,h,w,over", [
    (4, 4, 4, {}),                                  # planes of one block: the fifth tap has no column
    (4, 16, 4, dict(t_ref=100)),
    (4, 8, 8, {}),                                  # planes two blocks wide: most taps clamped
    (4, 24, 20, dict(t_ref=120, t_pred=120, subpel=False)),
    (4, 24, 20, dict(t_ref=1 << 20)),               # no reference block kept: no tiles at all
    (8, 40, 24, dict(t_ref=400)),
    (16, 64, 32, dict(t_ref=1500, win=8)),
    (64, 64, 64, {}),
])
def test_equal_to_per_ray_and_dense(block, h, w, over):
    import torch

    from paper_1902_09396_amd import lf

    enc = lfscene.get_config("tiny", block=block, **over)["enc"]
    stream = oracle.encode(crop_lf("tiny", 6, 5, h, w), enc)
    dense, sparse = lf.LightField(stream), lf.LightField(stream, sparse_refs=True)
    for cams in (lfscene.random_pinhole_cameras(5, 6, 5, w, h, 40, 21, seed=block),
                 lfscene.camera_path_orbit(13, 6, 5, w, h, 40, 21, radius=1.5)):
        dc = torch.from_numpy(cams).cuda()
        got = sparse.render_views(dc, 40, 21)
        assert torch.equal(got, sparse.render_views(dc, 40, 21, per_ray=True))
        assert torch.equal(got, dense.render_views(dc, 40, 21))
        for level in range(3):
            assert torch.equal(sparse.render_views_lod(level, dc, 40, 21), dense.render_views_lod(level, dc, 40, 21))
