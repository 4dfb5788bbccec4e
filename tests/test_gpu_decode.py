"""Random-access decoding, in request order and ordered by pixel block:
bit-exact against the oracle, clamped requests counted once."""

import ctypes as C

import numpy as np
import pytest


pytestmark = pytest.mark.gpu


def _requests(kind, n, nb, na, h, w, seed):
    rng = np.random.default_rng(seed)
    c = np.stack([rng.integers(0, nb, n), rng.integers(0, na, n), rng.integers(0, h, n), rng.integers(0, w, n)], 1)
    if kind == "rows":  # consecutive samples
        k = (np.arange(n) + 12345) % (nb * na * h * w)
        c = np.stack(np.unravel_index(k, (nb, na, h, w)), 1)
    elif kind == "one block":
        c[:, 2:] = c[:, 2:] % 16 + 32
    c = c.astype(np.int32)
    c[::97] += rng.integers(-300, 300, (len(c[::97]), 4)).astype(np.int32)  # outside the grid
    return c


@pytest.mark.parametrize("kind", ["random", "rows", "one block"])
@pytest.mark.parametrize("n", [1, 63, 65, 4097, 114687, 114688, 150001])
def test_orders_and_sizes(mid_stream, mid_oracle, kind, n):
    import torch

    from paper_1902_09396_amd import lf

    field, o = lf.LightField(mid_stream), mid_oracle
    dims = np.array([o.nb, o.na, o.h, o.w])
    need = C.c_int64()
    lf.check(lf.lib().lf_decode_workspace(field.handle, n, C.byref(need)))
    assert (need.value > 0) == (n >= 114688)
    coords = _requests(kind, n, *dims, seed=n)
    inside = np.clip(coords, 0, dims - 1)
    got = field.decode_pixels(torch.from_numpy(coords).cuda()).cpu().numpy()
    assert np.array_equal(got, o.decode_at(inside))
    assert field.clamped_coords() == int((coords != inside).any(1).sum())
    # the call without scratch
    out = torch.empty((n, 3), dtype=torch.uint8, device="cuda")
    dc = torch.from_numpy(coords).cuda()
    lf.check(lf.lib().lf_decode_pixels(field.handle, lf._ptr(dc), n, lf._ptr(out), lf._stream()))
    assert np.array_equal(out.cpu().numpy(), got)


def test_ordered_levels(mid_stream, mid_oracle):
    import torch

    from paper_1902_09396_amd import lf

    field, o = lf.LightField(mid_stream), mid_oracle
    for level in range(1, field.levels + 1):
        nb, na = -(-o.nb // (1 << level)), -(-o.na // (1 << level))
        coords = np.clip(_requests("random", 120000, nb, na, o.h, o.w, level), 0, np.array([nb, na, o.h, o.w]) - 1).astype(np.int32)
        got = field.decode_nodes(level, torch.from_numpy(coords).cuda()).cpu().numpy()
        assert np.array_equal(got, o.decode_node(level, coords))


def test_scratch_errors(mid_stream):
    import torch

    from paper_1902_09396_amd import lf

    field = lf.LightField(mid_stream)
    n = 114688
    dc = torch.zeros((n, 4), dtype=torch.int32, device="cuda")
    out = torch.empty((n, 3), dtype=torch.uint8, device="cuda")
    need = C.c_int64()
    lf.check(lf.lib().lf_decode_workspace(field.handle, n, C.byref(need)))
    ws = torch.empty(need.value, dtype=torch.uint8, device="cuda")
    call = lambda p, size: lf.lib().lf_decode_pixels_ordered(field.handle, 0, lf._ptr(dc), n, lf._ptr(out), p, size, lf._stream())  # noqa: E731
    assert call(lf._ptr(ws), need.value) == lf.LF_OK
    assert call(lf._ptr(ws), need.value - 1) == lf.LF_ENOMEM
    assert call(None, need.value) == lf.LF_EINVAL
    assert call(C.c_void_p(ws.data_ptr() + 16), need.value) == lf.LF_EINVAL
