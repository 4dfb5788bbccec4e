"""The encoder's four-pixel passes (colour with the first one or two hierarchy
levels, SRVs, block coding, payload packing) at the edges of their splits:
every block size they take, one to three tree levels (the fused hierarchy ends
at the root, below it, or is a single level), ragged clusters in either
direction, item counts that leave the last workgroup partly filled.  Streams
are integer data: every byte equals the oracle's."""

import numpy as np
import pytest

import lfscene
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block", [4, 8, 16, 32, 64])
@pytest.mark.parametrize("levels,nb,na", [(1, 2, 3), (2, 3, 3), (3, 5, 2), (3, 1, 6)])
def test_encode_quads(block, levels, nb, na):
    from paper_1902_09396_amd import lf

    rng = np.random.default_rng(block * 100 + levels * 10 + na)
    h, w = block, (3 if block < 64 else 1) * block
    base = rng.integers(0, 256, (1, 1, h, w, 3))
    x = np.clip(base + rng.integers(-40, 41, (nb, na, h, w, 3)), 0, 255).astype(np.uint8)
    x[nb - 1, na - 1] = 255 * (x[nb - 1, na - 1] > 127)
    enc = lfscene.get_config("tiny")["enc"]
    enc.update(levels=levels, block=block, step=[1 + 3 * l for l in range(levels)], win=[2 + l for l in range(levels)],
               t_ref=[block * 3] * levels, t_pred=[block * block] * levels)
    for over in ({}, {"no_mc": True}, {"zero_phase": True}):
        e = dict(enc, **over)
        got, exp = lf.encode(x, e), oracle.encode(x, e)
        assert got.size == exp.size and np.array_equal(got, exp), over
