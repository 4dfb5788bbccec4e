"""Unrelated views in long chunks take the plan for lone views, as in short ones."""

import numpy as np
import pytest

import lfscene
from conftest import lf_for

pytestmark = pytest.mark.gpu


def test_cost_of_many_unrelated_views():
    """48 unrelated 720p views, one chunk of 48 a tile, cost per view what 16
    do (20% more without the plan)."""
    import torch

    from paper_1902_09396_amd import lf

    light = np.tile(lf_for("tiny"), (3, 3, 8, 8, 1))[:17, :17]
    field = lf.LightField(lf.encode(np.ascontiguousarray(light), lfscene.get_config("path512")["enc"]))
    cams = torch.from_numpy(lfscene.random_pinhole_cameras(48, 17, 17, 512, 512, 1280, 720, 5)).cuda()
    times = []
    for n in (16, 48):
        best = float("inf")
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for first in range(0, 48, n):
                field.render_views(cams[first:first + n], 1280, 720)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        times.append(best)
    assert times[1] < 1.08 * times[0], times
