"""Loading: reference planes and the range checks, against the oracle."""

import numpy as np
import pytest

import lfscene
import oracle
from streamkit import Craft

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch

    assert torch.cuda.is_available()
    return torch


def _every_sample(na, nb, h, w):
    b, a, y, x = np.meshgrid(range(nb), range(na), range(h), range(w), indexing="ij")
    return np.stack([b, a, y, x], -1).reshape(-1, 4).astype(np.int32)


@pytest.mark.parametrize("block,h,w", [(1, 4, 6), (2, 6, 10), (4, 12, 20), (8, 24, 40), (16, 32, 48), (64, 64, 128)])
@pytest.mark.parametrize("amplitude", [0, 1, 9, 255])
def test_reference_planes(torch, block, h, w, amplitude):
    """Every sample of fields of noise coded losslessly: zero blocks, the
    narrowest and the widest value ranges of all three sequence families."""
    from paper_1902_09396_amd import lf

    rng = np.random.default_rng(block + amplitude)
    light = (rng.integers(0, amplitude + 1, (3, 3, h, w, 3)) * (rng.random((3, 3, 1, 1, 1)) < 0.8)).astype(np.uint8)
    enc = lfscene.get_config("tiny", block=block, step=1, win=2, no_mc=block == 1)["enc"]
    stream = oracle.encode(light, enc)
    field = lf.LightField(stream)
    coords = _every_sample(3, 3, h, w)
    got = field.decode_pixels(torch.from_numpy(coords).cuda()).cpu().numpy()
    assert np.array_equal(got, oracle.OracleLF(stream).decode_at(coords))
    assert np.array_equal(got.reshape(light.shape), light)


def test_sample_range_checked_by_decoding(torch):
    """Block modes wide enough that the table's bound exceeds the sample
    range, values that stay inside it: the load decodes every sample and
    accepts the stream, and every result equals the oracle's."""
    from paper_1902_09396_amd import lf

    k = Craft(na=4, nb=3, w=16, h=8, levels=2, block=4, step=[4, 4], win=[2, 2])
    rng = np.random.default_rng(8)
    k.root[0] = rng.integers(0, 256, k.root[0].shape)
    for l in range(2):
        for B in range(k.nb_l[l]):
            for A in range(k.na_l[l]):
                for blk in range(k.nblk):
                    if (A | B) & 1:  # 12-bit offsets from -100: up to (4095 - 100) * 4 as far as the table says
                        k.set_block_raw(0, l, B, A, blk, -100, 12, rng.integers(0, 200, 16))
                        k.set_mv(0, l, B, A, blk, int(rng.integers(-8, 9)), int(rng.integers(-8, 9)), 1)
                    else:
                        k.set_block(0, l, B, A, blk, rng.integers(-20, 20, 16))
    stream = k.build()
    o, field = oracle.OracleLF(stream), lf.LightField(stream)
    coords = _every_sample(4, 3, 8, 16)
    assert np.array_equal(field.decode_pixels(torch.from_numpy(coords).cuda()).cpu().numpy(), o.decode_at(coords))
    cams = lfscene.random_pinhole_cameras(3, 4, 3, 16, 8, 24, 16, seed=4, rho=0.25)
    dc = torch.from_numpy(cams).cuda()
    assert np.abs(field.render_views(dc, 24, 16).cpu().numpy() - o.render(cams, 24, 16)).max() <= 1e-5
    for level in range(3):
        got = field.render_views_lod(level, dc, 24, 16).cpu().numpy()
        assert np.abs(got - o.render_lod(level, cams, 24, 16)).max() <= 1e-5
