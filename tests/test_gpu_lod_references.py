"""Level-of-detail views that meet one reference node on a path of references
read its planes directly: the same pixels as the one-thread-per-ray decode,
among views that straddle nodes or meet predictive ones, in chunks of one to
many views; and such previews cost no more than others."""

import numpy as np
import pytest

import lfscene
import oracle
from conftest import crop_lf, lf_for

pytestmark = pytest.mark.gpu


def _cams(points, w, h, wo, ho):
    st = lfscene.cameras.full_frame_st(w, h, wo, ho)
    return np.stack([lfscene.cameras.fixed_uv_camera(u, v, st) for u, v in points])


@pytest.mark.parametrize("sparse", [False, True])
@pytest.mark.parametrize("block", [4, 16])
@pytest.mark.parametrize("views", [1, 3, 4, 5, 40])
def test_pixels(block, sparse, views):
    import torch

    from paper_1902_09396_amd import lf

    levels = 3
    cfg = lfscene.get_config("tiny", levels=levels, step=[4] * levels, win=[4] * levels, t_ref=[0] * levels,
                             t_pred=[0] * levels, block=block)
    stream = oracle.encode(crop_lf("tiny", 8, 7, 32, 48), cfg["enc"])
    o, field = oracle.OracleLF(stream), lf.LightField(stream, sparse_refs=sparse)
    rng = np.random.default_rng(views)
    # views inside the first node, across its border, inside others, at the grid's corners
    points = [(0.5, 0.5), (1.5, 0.2), (0.3, 5.9), (7.0, 6.0), (4.4, 4.1), (2.5, 0.5), (0.0, 0.0)]
    points = [points[k % 7] if k < 14 else tuple(rng.uniform(0, 7, 2)) for k in range(views)]
    for wo, ho in ((48, 32), (45, 19), (100, 70)):
        cams = _cams(points, 48, 32, wo, ho)
        dc = torch.from_numpy(cams).cuda()
        for level in range(levels + 1):
            got = field.render_views_lod(level, dc, wo, ho).cpu().numpy()
            assert np.abs(got - o.render_lod(level, cams, wo, ho)).max() <= 1e-5, (level, wo)


def test_cost_of_one_reference():
    """From a point inside a reference node against a point inside a predictive
    one, level 1 of 2: twelve plane reads a ray, so no dearer (four times
    cheaper; it was as dear through the tile stages)."""
    import torch

    from paper_1902_09396_amd import lf

    enc = lfscene.get_config("tiny", levels=2, step=[4] * 2, win=[4] * 2, t_ref=[0] * 2, t_pred=[0] * 2, block=8)["enc"]
    light = np.tile(lf_for("tiny"), (2, 2, 4, 4, 1))[:9, :9]
    field = lf.LightField(lf.encode(np.ascontiguousarray(light), enc))
    times = []
    for u in (0.5, 2.5):
        dc = torch.from_numpy(_cams([(u, u), (u + 0.01, u)], 256, 256, 986, 429)).cuda()
        run = lambda: field.render_views_lod(1, dc, 986, 429)  # noqa: E731
        best = float("inf")
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                run()
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        times.append(best)
    assert times[0] < 0.7 * times[1], times


@pytest.mark.parametrize("na,nb,levels", [(8, 8, 3), (17, 9, 4), (8, 4, 3)])
def test_level_below_the_root_by_views(na, nb, levels):
    """40 views in one call (five and more a workgroup: tiles, except over a
    single row of nodes) and in calls of four (one thread per ray)."""
    import torch

    from paper_1902_09396_amd import lf

    cfg = lfscene.get_config("tiny", levels=levels, step=[4] * levels, win=[4] * levels, t_ref=[0] * levels,
                             t_pred=[0] * levels, block=8)
    light = np.tile(lf_for("tiny"), (2, 3, 1, 1, 1))[:nb, :na]
    field = lf.LightField(lf.encode(np.ascontiguousarray(light), cfg["enc"]))
    wo, ho = 512, 128
    assert lf.render_config(40, wo, ho)[1] >= 5 > lf.render_config(4, wo, ho)[1]
    cams = np.concatenate([lfscene.camera_path_orbit(20, na, nb, 64, 64, wo, ho, radius=1.2),
                           lfscene.random_pinhole_cameras(20, na, nb, 64, 64, wo, ho, seed=na)])
    dc = torch.from_numpy(cams).cuda()
    got = field.render_views_lod(levels - 1, dc, wo, ho)
    assert torch.equal(got, torch.cat([field.render_views_lod(levels - 1, dc[k:k + 4], wo, ho) for k in range(0, 40, 4)]))
