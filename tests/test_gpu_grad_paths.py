"""The adjoint's kernels at the sizes where their paths change, against the oracle.

Tolerances are those of the FP32 adjoint against the oracle's FP64 reverse
mode: 1e-3 of each element plus 1e-6 (residuals) or 1e-5 (shifts) of the
largest one.
"""

import ctypes as C

import numpy as np
import pytest

import lfscene
import oracle
from conftest import crop_lf

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch

    assert torch.cuda.is_available()
    return torch


def _field(na, nb, h, w, block, levels=2, **enc):
    from paper_1902_09396_amd import lf

    cfg = lfscene.get_config("tiny", levels=levels, step=[4] * levels, win=[4] * levels, t_ref=[0] * levels,
                             t_pred=[0] * levels, block=block, **enc)
    stream = oracle.encode(crop_lf("tiny", na, nb, h, w), cfg["enc"])
    return oracle.OracleLF(stream), lf.LightField(stream)


def _params(torch, field, seed, spread):
    rng = np.random.default_rng(seed)
    res, sh = field.export_params()
    far = sh.cpu().numpy() + rng.uniform(-spread, spread, size=tuple(sh.shape)).astype(np.float32)
    return rng, res, torch.from_numpy(far.astype(np.float32)).cuda()


def _compare(o, res, sh, cams, wo, ho, g, got_r, got_s):
    o_r, o_s = o.relaxed_grad(res.cpu().numpy(), sh.cpu().numpy(), cams, wo, ho, g.astype(np.float64))
    got_r, got_s = got_r.cpu().numpy().astype(np.float64), got_s.cpu().numpy().astype(np.float64)
    for got, ref, floor in ((got_r, o_r, 1e-6), (got_s, o_s, 1e-5)):
        err = np.abs(got - ref)
        assert np.all(err <= 1e-3 * np.abs(ref) + floor * np.abs(ref).max() + 1e-12), err.max()


@pytest.mark.parametrize("block,h,w,views", [(1, 5, 7, 2), (4, 28, 36, 1), (8, 40, 48, 2), (16, 48, 32, 1), (32, 32, 64, 2)])
def test_reference_and_shift_passes(torch, block, h, w, views):
    """Blocks of one pixel, of one to several lanes' quads and of several
    rounds of a wave; planes that are not whole 16x16 tiles; one view only,
    which leaves most blocks without a gradient."""
    o, field = _field(5, 3, h, w, block, no_mc=block == 1)
    rng, res, sh = _params(torch, field, block, 3.0)
    cams = lfscene.random_pinhole_cameras(views, 5, 3, w, h, 21, 17, seed=block)
    g = rng.normal(size=(views, 3, 17, 21)).astype(np.float32)
    got = field.render_backward(res, sh, torch.from_numpy(cams).cuda(), 21, 17, torch.from_numpy(g).cuda())
    _compare(o, res, sh, cams, 21, 17, g, *got)


def test_gradient_buffer_alignment(torch):
    """A gradient buffer that is not 16-byte aligned gives the same gradients."""
    from paper_1902_09396_amd import lf

    o, field = _field(4, 3, 32, 48, 8)
    rng, res, sh = _params(torch, field, 7, 1.0)
    cams = lfscene.random_pinhole_cameras(2, 4, 3, 48, 32, 30, 20, seed=3)
    g = rng.normal(size=(2, 3, 20, 30)).astype(np.float32)
    dc, dg = torch.from_numpy(cams).cuda(), torch.from_numpy(g).cuda()
    need = C.c_int64()
    lf.check(lf.lib().lf_backward_workspace(field.handle, 2, 30, 20, C.byref(need)))
    ws = torch.empty(need.value, dtype=torch.uint8, device="cuda")
    buf = torch.empty(res.numel() + 1, device="cuda")
    g_res, g_sh = buf[1:].view(res.shape), torch.empty_like(sh)
    lf.check(lf.lib().lf_render_backward(field.handle, lf._ptr(res), lf._ptr(sh), lf._ptr(dc), 2, 30, 20, lf._ptr(dg),
                                         lf._ptr(g_res), lf._ptr(g_sh), lf._ptr(ws), need.value, lf._stream()))
    _compare(o, res, sh, cams, 30, 20, g, g_res, g_sh)


def _cams(kind, views, na, nb, w, h, wo, ho):
    """Separable cameras (diagonal homographies, some mirrored), projective
    ones, or both in one batch."""
    cams = lfscene.random_pinhole_cameras(views, na, nb, w, h, wo, ho, seed=wo)
    for c in cams[::3]:  # mirrored: coordinates fall along the row
        c[2], c[0] = c[2] + c[0] * wo, -c[0]
        c[11], c[9] = c[11] + c[9] * wo, -c[9]
    if kind != "separable":
        warped = lfscene.projective_warp(cams, 3e-3, -2e-3)
        cams = warped if kind == "projective" else np.where(np.arange(views)[:, None] % 2 == 0, cams, warped)
    return np.ascontiguousarray(cams, dtype=np.float32)


@pytest.mark.parametrize("kind", ["separable", "projective", "mixed"])
@pytest.mark.parametrize("na,nb,levels,wo,ho,views", [(5, 3, 1, 33, 7, 3), (6, 7, 2, 64, 40, 4), (5, 5, 3, 9, 70, 3),
                                                      (8, 8, 4, 40, 30, 2), (3, 4, 2, 2, 1, 5)])
def test_gather_paths(torch, kind, na, nb, levels, wo, ho, views):
    """Sample gradients from the axis tables, from sorted records and from
    both, for every depth of the fused tree; frames of 2x1 pixels are too
    small for the tables and always take the records."""
    o, field = _field(na, nb, 48, 40, 8, levels)
    rng, res, sh = _params(torch, field, levels, 0.25)
    cams = _cams(kind, views, na, nb, 40, 48, wo, ho)
    g = rng.normal(size=(views, 3, ho, wo)).astype(np.float32)
    args = (res, sh, torch.from_numpy(cams).cuda(), wo, ho, torch.from_numpy(g).cuda())
    got = field.render_backward(*args)
    _compare(o, res, sh, cams, wo, ho, g, *got)
    again = field.render_backward(*args)
    assert all(torch.equal(x, y) for x, y in zip(got, again))


def test_record_sort_large(torch):
    """More records than one workgroup's round of the sort (projective views
    of 256x256), magnified so that many records share a key."""
    o, field = _field(4, 4, 32, 32, 8)
    rng, res, sh = _params(torch, field, 5, 0.25)
    cams = _cams("projective", 3, 4, 4, 32, 32, 256, 256)
    g = rng.normal(size=(3, 3, 256, 256)).astype(np.float32)
    got = field.render_backward(res, sh, torch.from_numpy(cams).cuda(), 256, 256, torch.from_numpy(g).cuda())
    _compare(o, res, sh, cams, 256, 256, g, *got)


@pytest.mark.parametrize("block,wo,ho,warp", [(8, 37, 19, 0.0), (8, 24, 24, 0.0), (8, 8, 6, 0.0), (2, 33, 9, 0.0),
                                              (16, 40, 40, 4e-3), (8, 1, 1, 0.0)])
def test_relaxed_forward_tiles(torch, block, wo, ho, warp):
    """Tiles staged whole, in four parts and ray by ray (frames ever smaller
    than the captured views), ragged sizes and projective cameras: within 1e-5
    of the oracle, as every forward."""
    o, field = _field(8, 8, 64, 64, block)
    _, res, sh = _params(torch, field, wo, 2.0)
    cams = lfscene.random_pinhole_cameras(3, 8, 8, 64, 64, wo, ho, seed=block, zoom_range=(0.9, 1.0))
    if warp:
        cams = lfscene.projective_warp(cams, warp, -warp)
    got = field.render_relaxed(res, sh, torch.from_numpy(cams).cuda(), wo, ho).cpu().numpy().astype(np.float64)
    assert np.abs(got - o.render_relaxed(res.cpu().numpy(), sh.cpu().numpy(), cams, wo, ho)).max() <= 1e-5
