"""Quarter-pel refinement of 12-bit values (two pixels per packed 16-bit
instruction) against the oracle: values at both ends of [-2048, 2047], where
16 v + 8 just fits 16 bits, and one step beyond in a few windows or blocks,
which take the general refinement; windows small enough that the best integer
displacement and its neighbourhood reach the search limits on every side."""

import numpy as np
import pytest

from test_gpu_search import _all_items, _expect, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bs,win", [(2, 1), (2, 4), (4, 1), (4, 6), (8, 1), (8, 5), (16, 1), (16, 8), (32, 3), (64, 2)])
@pytest.mark.parametrize("beyond", [False, True])
def test_search_narrow(bs, win, beyond):
    import torch

    rng = np.random.default_rng(7 * bs + win)
    n, h, w = 3, max(2 * bs, 32), max(2 * bs, 48) // bs * bs
    ref = rng.integers(-2048, 2048, (n, h, w))
    ref[0] = rng.choice([-2048, 2047], (h, w))
    y, x = np.mgrid[0:h, 0:w]
    pred = np.empty_like(ref)
    for p in range(n):  # shifted by a fraction, the phase of every other plane negated
        dy, dx = rng.integers(-win, win + 1, 2)
        a = ref[p][np.clip(y + dy, 0, h - 1), np.clip(x + dx, 0, w - 1)]
        b = ref[p][np.clip(y + dy + 1, 0, h - 1), np.clip(x + dx - 1, 0, w - 1)]
        pred[p] = (-1) ** p * ((3 * a + b) // 4)
    pred = np.clip(pred, -2048, 2047)
    if beyond:
        ref[1, h // 2, w // 2], pred[2, 0, 0], pred[0, h - 1, w - 1] = 2048, -2049, 2048
    pred, ref = pred.astype(np.int16), ref.astype(np.int16)
    items = _all_items(n, h, w, bs, rng)
    items[::2, 1] = items[::2, 0]
    if len(items) > 120:
        items = items[rng.choice(len(items), 120, replace=False)]
    assert np.array_equal(_run(torch, pred, ref, items, bs, win), _expect(pred, ref, items, bs, win))
