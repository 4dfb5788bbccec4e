"""The adjoint's gather over small and large fields, few and many rays: results
against the oracle's FP64 reverse mode (1e-3 of each element plus 1e-6, for
shifts 1e-5, of the largest), and no form of it many times dearer than another."""

import numpy as np
import pytest

import lfscene
import oracle
from conftest import lf_for

pytestmark = pytest.mark.gpu


def _stream(na, nb, h, w, block, levels):
    light = np.tile(lf_for("tiny"), (2, 2, -(-h // 64), -(-w // 64), 1))[:nb, :na, :h, :w]
    cfg = lfscene.get_config("tiny", levels=levels, step=[4] * levels, win=[4] * levels, t_ref=[0] * levels,
                             t_pred=[0] * levels, block=block)
    return oracle.encode(np.ascontiguousarray(light), cfg["enc"])


def _cams(kind, views, na, nb, w, h, wo, ho):
    cams = lfscene.random_pinhole_cameras(views, na, nb, w, h, wo, ho, seed=wo)
    if kind == "mixed":
        warped = lfscene.projective_warp(cams, 0.2 / wo, -0.1 / ho)
        cams = np.where(np.arange(views)[:, None] % 2 == 0, cams, warped)
    return np.ascontiguousarray(cams, dtype=np.float32)


def _compare(field, o, cams, wo, ho, seed):
    import torch

    rng = np.random.default_rng(seed)
    res, sh = field.export_params()
    sh = sh + torch.from_numpy(rng.uniform(-0.25, 0.25, tuple(sh.shape)).astype(np.float32)).cuda()
    g = rng.normal(size=(len(cams), 3, ho, wo)).astype(np.float32)
    got = field.render_backward(res, sh, torch.from_numpy(cams).cuda(), wo, ho, torch.from_numpy(g).cuda())
    ref = o.relaxed_grad(res.cpu().numpy(), sh.cpu().numpy(), cams, wo, ho, g.astype(np.float64))
    for x, y, floor in zip(got, ref, (1e-6, 1e-5)):
        err = np.abs(x.cpu().numpy().astype(np.float64) - y)
        assert np.all(err <= 1e-3 * np.abs(y) + floor * np.abs(y).max() + 1e-12), err.max()


def _time(f):
    import torch

    best = float("inf")
    for _ in range(4):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        f()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


@pytest.mark.parametrize("kind", ["separable", "mixed"])
@pytest.mark.parametrize("na,nb,h,w,levels,views,wo,ho", [
    (9, 9, 192, 208, 3, 2, 40, 30),  # enough clusters for the chip and few rays: two levels in registers
    (9, 9, 112, 96, 2, 2, 40, 30),  # one level
    (9, 9, 112, 96, 2, 1, 700, 500), (13, 9, 192, 208, 3, 1, 1100, 700),  # leaves ahead of the sums where records are gathered
    (9, 9, 192, 208, 3, 1, 1200, 800),  # more records than a quarter of the samples
    (5, 3, 64, 48, 4, 2, 20, 30)])  # few clusters
def test_levels_in_registers(kind, na, nb, h, w, levels, views, wo, ho):
    from paper_1902_09396_amd import lf

    s = _stream(na, nb, h, w, 16, levels)
    _compare(lf.LightField(s), oracle.OracleLF(s), _cams(kind, views, na, nb, w, h, wo, ho), wo, ho, levels)


def test_tree_height_of_a_small_field():
    """Levels summed in registers take threads from a small field: a taller
    tree costs about what a flat one does (4.5 times it with two levels)."""
    import torch

    from paper_1902_09396_amd import lf

    cams = lfscene.projective_warp(lfscene.random_pinhole_cameras(2, 5, 5, 64, 64, 1280, 720, seed=1), 2e-4, -1e-4)
    dc = torch.from_numpy(cams).cuda()
    g = torch.ones(2, 3, 720, 1280, device="cuda")
    times = []
    for levels in (1, 3):
        field = lf.LightField(_stream(5, 5, 64, 64, 8, levels))
        res, sh = field.export_params()
        times.append(_time(lambda: field.render_backward(res, sh, dc, 1280, 720, g)))
    assert times[1] < 2 * times[0], times


def _wide(views, n, h, wo):
    """Separable views that each span every light-field view of an n x n grid."""
    return lfscene.random_pinhole_cameras(views, n, n, h, h, wo, wo, seed=5, ez_range=(-9.0, -8.0), zoom_range=(0.95, 1.0))


@pytest.mark.parametrize("views,warped", [(10, 0), (24, 0), (24, 5)])
def test_small_frames_over_many_views(views, warped):
    """Enough of them that the tables would be walked mostly for nothing: all
    go by records (from 17 views on; with 10 the tables serve)."""
    from paper_1902_09396_amd import lf

    s = _stream(9, 9, 192, 192, 16, 3)
    cams = _wide(views, 9, 192, 13)
    if warped:
        cams[:warped] = lfscene.projective_warp(cams[:warped], 1e-2, -5e-3)
    _compare(lf.LightField(s), oracle.OracleLF(s), cams, 13, 13, views)


def test_cost_of_small_frames_over_many_views():
    """Views over the whole grid cost about what views from one point each do
    (six times that when every sample walks every view)."""
    import torch

    from paper_1902_09396_amd import lf

    light = np.tile(lf_for("tiny"), (3, 3, 4, 4, 1))[:17, :17]
    field = lf.LightField(lf.encode(np.ascontiguousarray(light), lfscene.get_config("path512")["enc"]))
    res, sh = field.export_params()
    g = torch.ones(400, 3, 32, 32, device="cuda")
    times = []
    for cams in (lfscene.random_fixed_uv_cameras(400, 17, 17, 256, 256, 32, 32, 5), _wide(400, 17, 256, 32)):
        dc = torch.from_numpy(cams).cuda()
        times.append(_time(lambda: field.render_backward(res, sh, dc, 32, 32, g)))
    assert times[1] < 3 * times[0], times
