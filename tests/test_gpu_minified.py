"""Far minified views, whose tiles all exceed the LDS budget and are rendered
ray by ray, one thread per channel: the same pixels as the one-thread-per-ray
kernel.  Tile counts below and above the pass's grid, odd frame sizes (part
tiles), and enough tiles that a workgroup checks more than it has threads."""

import numpy as np
import pytest

import lfscene
import oracle
from conftest import crop_lf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block,residency,n,wo,ho", [
    (16, "dense", 1, 33, 9), (16, "dense", 300, 32, 8), (16, "dense", 193000, 32, 8), (4, "dense", 90, 35, 17),
    (8, "sparse", 40, 31, 7), (8, "420", 40, 40, 11), (16, "420", 260, 32, 8)])
def test_minified(block, residency, n, wo, ho):
    import torch

    from paper_1902_09396_amd import lf

    enc = lfscene.get_config("tiny")["enc"]
    enc.update(block=block, chroma420=residency == "420")
    field = lf.LightField(oracle.encode(crop_lf("tiny", 7, 6, 64, 64), enc), sparse_refs=residency == "sparse")
    cams = lfscene.random_pinhole_cameras(min(n, 97), 7, 6, 64, 64, wo, ho, seed=n)
    cams = torch.from_numpy(cams[np.arange(n) % len(cams)]).cuda()
    assert torch.equal(field.render_views(cams, wo, ho), field.render_views(cams, wo, ho, per_ray=True))
