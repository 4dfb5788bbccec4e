"""Level-of-detail renders through the tile kernel, every level, against the
oracle (1e-5, as every integer-decode render)."""

import numpy as np
import pytest

import lfscene
import oracle
from conftest import crop_lf

pytestmark = pytest.mark.gpu


def _cams(kind, na, nb, w, h, wo, ho):
    if kind == "orbit":  # one st window: the shared (s, t) sums across views
        return lfscene.camera_path_orbit(14, na, nb, w, h, wo, ho, radius=1.2)
    cams = lfscene.random_pinhole_cameras(5, na, nb, w, h, wo, ho, seed=na)
    return lfscene.projective_warp(cams, 2e-3, 1e-3) if kind == "projective" else cams


@pytest.mark.parametrize("chroma420", [False, True])
@pytest.mark.parametrize("kind", ["orbit", "pinhole", "projective"])
@pytest.mark.parametrize("na,nb,levels,block", [(8, 7, 3, 16), (5, 8, 2, 8), (3, 3, 2, 4), (8, 8, 4, 16)])
def test_every_level(na, nb, levels, block, kind, chroma420):
    import torch

    from paper_1902_09396_amd import lf

    cfg = lfscene.get_config("tiny", levels=levels, step=[4] * levels, win=[4] * levels, t_ref=[0] * levels,
                             t_pred=[0] * levels, block=block)
    cfg["enc"]["chroma420"] = chroma420
    stream = oracle.encode(crop_lf("tiny", na, nb, 64, 32), cfg["enc"])
    o, field = oracle.OracleLF(stream), lf.LightField(stream)
    cams = _cams(kind, na, nb, 32, 64, 45, 50)
    dc = torch.from_numpy(cams).cuda()
    for level in range(levels + 1):
        got = field.render_views_lod(level, dc, 45, 50).cpu().numpy()
        assert np.abs(got - o.render_lod(level, cams, 45, 50)).max() <= 1e-5, level
    assert torch.equal(field.render_views_lod(0, dc, 45, 50), field.render_views(dc, 45, 50, per_ray=True))
