"""Random-access decoding of fields too small to be ordered: bit-exact against
the oracle on both sides of the line between the two kernels, and no jump in
cost where larger fields begin to be ordered."""

import numpy as np
import pytest

import oracle
from conftest import lf_for, stream_for

pytestmark = pytest.mark.gpu


def _decode(lf, torch, field, coords):
    out = torch.empty((coords.shape[0], 3), dtype=torch.uint8, device="cuda")
    lf.check(lf.lib().lf_decode_pixels(field.handle, lf._ptr(coords), coords.shape[0], lf._ptr(out), lf._stream()))
    return out


@pytest.mark.parametrize("n", [114687, 114688, 163839, 163840])
@pytest.mark.parametrize("block", [2, 8])
def test_both_kernels(block, n):
    import torch

    from paper_1902_09396_amd import lf

    s = stream_for("tiny", lf_for("tiny"), block=block)
    o, field = oracle.OracleLF(s), lf.LightField(s)
    rng = np.random.default_rng(n)
    coords = np.stack([rng.integers(0, m, n) for m in (8, 8, 64, 64)], 1).astype(np.int32)
    dc = torch.from_numpy(coords).cuda()
    expect = o.decode_at(coords)
    assert np.array_equal(_decode(lf, torch, field, dc).cpu().numpy(), expect)
    assert np.array_equal(field.decode_pixels(dc).cpu().numpy(), expect)


def test_cost_of_one_more_request():
    """114,688 consecutive requests against 114,687 (twice the time where the
    larger call went to the other kernel)."""
    import torch

    from paper_1902_09396_amd import lf

    light = np.tile(lf_for("tiny"), (2, 2, 2, 2, 1))[:16, :16, :96, :96]
    enc = {"levels": 4, "block": 16, "step": [4] * 4, "win": [8] * 4, "t_ref": [0] * 4, "t_pred": [0] * 4, "subpel": True}
    field = lf.LightField(lf.encode(np.ascontiguousarray(light), enc))
    k = torch.arange(114688)
    x, k = k % 96, k // 96
    y, k = k % 96, k // 96
    coords = torch.stack([k // 16, k % 16, y, x], 1).to(torch.int32).cuda()
    times = []
    for n in (114687, 114688):
        part, best = coords[:n].contiguous(), float("inf")
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(50):
                _decode(lf, torch, field, part)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        times.append(best)
    assert times[1] < 1.4 * times[0], times
