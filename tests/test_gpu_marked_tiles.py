"""Tiles whose box of captured pixels alone exceeds the tile renderer's budget,
checked on the host, are rendered by the pass over marked tiles: the pixels of
the one-thread-per-ray kernel, in launches smaller and larger than that pass's
grid, with the first row of tiles marked in every view and in every third."""

import numpy as np
import pytest

import lfscene
import oracle
from conftest import lf_for

pytestmark = pytest.mark.gpu


def _boxes(torch, lf, dc, wo, ho):
    """Captured pixels in the box of every tile: [views, tiles]."""
    st = lf.ray_coords(dc, wo, ho)[..., 2:].cpu().numpy()
    k = np.clip(np.floor(st), 0, 126)
    out = []
    for y in range(0, ho, 8):
        for x in range(0, wo, 32):
            t = k[:, y:y + 8, x:x + 32].reshape(len(k), -1, 2)
            out.append((t.max(1) - t.min(1) + 2).prod(1))
    return np.stack(out, 1)


@pytest.mark.parametrize("every", [1, 3])
@pytest.mark.parametrize("block,residency,views,wo,ho", [
    (16, "dense", 3, 33, 9), (16, "dense", 400, 32, 8), (4, "dense", 40, 35, 17), (8, "dense", 700, 32, 16),
    (8, "sparse", 300, 31, 8), (8, "420", 300, 32, 8)])
def test_marked(block, residency, views, wo, ho, every):
    import torch

    from paper_1902_09396_amd import lf

    enc = lfscene.get_config("tiny", block=block)["enc"]
    enc["chroma420"] = residency == "420"
    light = np.ascontiguousarray(np.tile(lf_for("tiny"), (1, 1, 2, 2, 1))[:6, :7])
    field = lf.LightField(oracle.encode(light, enc), sparse_refs=residency == "sparse")
    far = lfscene.random_pinhole_cameras(views, 7, 6, 128, 128, wo, ho, seed=block, zoom_range=(0.98, 1.0))
    near = lfscene.random_pinhole_cameras(views, 7, 6, 128, 128, wo, ho, seed=block, zoom_range=(0.15, 0.2))
    for cams, rows in ((far, 14.0), (near, 2.0)):  # captured rows per output row
        cams[:, 13], cams[:, 14] = rows, -0.5
    pick = np.arange(views) % every == 0
    dc = torch.from_numpy(np.where(pick[:, None], far, near).astype(np.float32)).cuda()
    box = _boxes(torch, lf, dc, wo, ho)[:, :wo // 32]
    budget = 4096 if block == 16 else 6144
    assert (box[pick] > budget).all() and (every == 1 or (box[~pick] < budget).all())
    assert torch.equal(field.render_views(dc, wo, ho), field.render_views(dc, wo, ho, per_ray=True))
