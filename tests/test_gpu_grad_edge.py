"""The adjoint at the edges of what it accepts, against the oracle's FP64
reverse mode (1e-3 of each element plus 1e-6, for shifts 1e-5, of the largest)."""

import numpy as np
import pytest

import lfscene
import oracle
from streamkit import Craft

pytestmark = pytest.mark.gpu


def _close(got, ref, floor):
    got = got.cpu().numpy().astype(np.float64)
    return np.all(np.abs(got - ref) <= 1e-3 * np.abs(ref) + floor * np.abs(ref).max() + 1e-12)


def _aligned(stream):
    """The sections after the root moved to a multiple of 4 bytes."""
    off = stream[112:176].copy().view(np.uint64)  # (offset, size) of root, table, payload, motion
    end = int(off[0] + off[1])
    pad = -end % 4
    off[2::2] += pad
    return np.concatenate([stream[:112], off.view(np.uint8), stream[176:end], np.zeros(pad, np.uint8), stream[end:]])


def _noise(na, nb, w, h, levels, block, seed):
    k = Craft(na=na, nb=nb, w=w, h=h, levels=levels, block=block, step=[3] * levels, win=[2] * levels)
    rng = np.random.default_rng(seed)
    k.root[:] = rng.integers(-60, 200, k.root.shape)
    for c in range(3):
        for l in range(levels):
            for B in range(k.nb_l[l]):
                for A in range(k.na_l[l]):
                    for blk in range(k.nblk):
                        k.set_block(c, l, B, A, blk, rng.integers(-9, 10, block * block))
                        if (A | B) & 1:
                            k.set_mv(c, l, B, A, blk, *(int(v) for v in rng.integers(-8, 9, 2)), int(rng.integers(-1, 2)))
    return _aligned(k.build())


@pytest.mark.parametrize("na,nb,levels", [(2, 1, 1), (1, 2, 1), (4, 4, 2), (5, 3, 3)])
@pytest.mark.parametrize("w,h", [(1, 1), (2, 1), (1, 2), (1, 5)])
def test_planes_of_one_pixel_wide_blocks(na, nb, levels, w, h):
    """1x1 blocks on the smallest planes: two taps of a row are read together,
    and the last predictive plane ends where the gradient buffer does."""
    import torch

    from paper_1902_09396_amd import lf

    stream = _noise(na, nb, w, h, levels, 1, seed=10 * na + w)
    o, field = oracle.OracleLF(stream), lf.LightField(stream)
    rng = np.random.default_rng(na + h)
    res, sh = field.export_params()
    sh = sh + torch.from_numpy(rng.uniform(-1.5, 1.5, tuple(sh.shape)).astype(np.float32)).cuda()
    cams = lfscene.random_pinhole_cameras(2, na, nb, w, h, 6, 5, seed=w, rho=0.3)
    g = rng.normal(size=(2, 3, 5, 6)).astype(np.float32)
    got = field.render_backward(res, sh, torch.from_numpy(cams).cuda(), 6, 5, torch.from_numpy(g).cuda())
    ref = o.relaxed_grad(res.cpu().numpy(), sh.cpu().numpy(), cams, 6, 5, g.astype(np.float64))
    assert _close(got[0], ref[0], 1e-6) and _close(got[1], ref[1], 1e-5)


def _shifted(torch, wo, ho, seed=5, levels=1, w=48, h=32):
    """A 2x2 field whose views are all rendered, its parameters with small
    shifts, and the record of block `blk` of channel 0, view (b, a)."""
    from paper_1902_09396_amd import lf

    stream = _noise(2, 2, w, h, levels, 8, seed)
    field = lf.LightField(stream)
    res, sh = field.export_params()
    st = lfscene.cameras.full_frame_st(w, h, wo, ho)
    cams = np.stack([lfscene.cameras.fixed_uv_camera(u, v, st) for u, v in ((0.4, 0.3), (0.7, 0.6))])
    nblk = (w // 8) * (h // 8)
    code = {(0, 1): 0, (1, 0): 1, (1, 1): 2}
    return oracle.OracleLF(stream), field, res, sh, torch.from_numpy(cams).cuda(), lambda b, a, blk: code[b, a] * nblk + blk


@pytest.mark.parametrize("wo,ho", [(48, 32), (8, 8)])  # tiles staged in LDS, and ray by ray
@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("value", [1e6, -1e6, 3e9, -3e9, 3e38, np.inf, -np.inf, np.nan])
def test_forward_of_any_shift(value, axis, wo, ho):
    """Shifts past every integer and no number at all: finite ones read the
    border sample, the others make their block's own samples NaN and no more."""
    import torch

    _, field, res, sh, cams, rec = _shifted(torch, wo, ho)
    changed, limit = sh.clone(), sh.clone()
    for blk in (0, 5, 23):
        for view in ((0, 1), (1, 0), (1, 1)):
            changed[rec(*view, blk), axis] = value
            limit[rec(*view, blk), axis] = 1000.0 if value > 0 else -1000.0
    got = field.render_relaxed(res, changed, cams, wo, ho)
    ref = field.render_relaxed(res, limit, cams, wo, ho)
    if np.isfinite(value):
        assert torch.equal(got, ref)
    else:
        bad = torch.isnan(got)
        assert bad.any() and torch.equal(got[~bad], ref[~bad])
        same = field.render_relaxed(res, sh, cams, wo, ho)
        assert torch.equal(same[~bad], got[~bad])  # rays that read no changed block


@pytest.mark.parametrize("axis", [0, 1])
def test_backward_of_a_nan_shift(axis):
    """The taps of a NaN shift count as clamped to the first column (row), as
    those of a shift far beyond it: NaN in the gradients of the reference's
    pixels there and of the block's shift, and nowhere else."""
    import torch

    _, field, res, sh, cams, rec = _shifted(torch, 48, 32, seed=6)
    g = torch.ones(2, 3, 32, 48, device="cuda")
    far = sh.clone()
    base = field.render_backward(res, sh, cams, 48, 32, g)
    k = next(rec(*view, 0) for view in ((0, 1), (1, 0), (1, 1)) if base[1][rec(*view, 0)].any())  # a block with a phase
    far[k, axis] = -1000.0
    ref = field.render_backward(res, far, cams, 48, 32, g)
    far[k, axis] = float("nan")
    got = field.render_backward(res, far, cams, 48, 32, g)
    bad = torch.isnan(got[0])
    where = torch.zeros_like(bad)  # reference node: the first of the four of level 0
    # along the other axis: eight pixels, a shift of at most two and the second tap
    (where[0, 0, :11, 0] if axis == 0 else where[0, 0, 0, :11])[:] = True
    assert bad.any() and not (bad & ~where).any()
    assert torch.isnan(got[1][k]).any() and not torch.isnan(torch.cat([got[1][:k], got[1][k + 1:]])).any()
    assert torch.allclose(got[0][~where], ref[0][~where], rtol=1e-5, atol=1e-7)
