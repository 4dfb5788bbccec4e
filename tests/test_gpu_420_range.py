"""4:2:0 handles whose value range the block table and the vector sequences
leave open: the load decides by the values, the tile renderer serves those that
fit its 16-bit lanes, and the others are rendered one thread per ray.  Nothing
is refused, and every pixel is the oracle's (1e-5)."""

import ctypes as C

import numpy as np
import pytest

import lfscene
import oracle
from conftest import lf_for
from streamkit import pack_plain

pytestmark = pytest.mark.gpu

BLOCK, LEVELS = 8, 2
WO, HO = 333, 217


def _base():
    enc = lfscene.get_config("tiny", block=BLOCK, levels=LEVELS)["enc"]
    enc["chroma420"] = True
    return oracle.encode(lf_for("tiny"), enc)


def _unpack(words, mode, n):
    w = np.concatenate([words, np.zeros(4, np.uint32)]).astype(np.uint32)
    out = np.zeros(n, np.uint32)
    oracle.lib().orc_bise_unpack(w.ctypes.data_as(C.c_void_p), int(mode), int(n), out.ctypes.data_as(C.c_void_p))
    return out


class _Stream:
    """The sections of a stream, to be changed and put together again."""

    def __init__(self, s):
        off = s[112:176].copy().view(np.uint64).astype(int)
        self.head = s[:1024].copy()
        self.root, self.table, self.payload, self.mv = (s[off[k]:off[k] + off[k + 1]].copy() for k in (0, 2, 4, 6))
        self.payload, self.mv = self.payload.view(np.uint32), self.mv.view(np.uint32)

    def build(self):
        parts = [self.root, self.table, self.payload.view(np.uint8), self.mv.view(np.uint8)]
        at, off = 1024, []
        for p in parts:
            off += [at, p.size]
            at += p.size
        self.head[112:176] = np.array(off, np.uint64).view(np.uint8)
        return np.concatenate([self.head] + parts)

    def widen_block(self):
        """A block's values again, in a 13-bit sequence."""
        t = self.table.reshape(-1, 8)
        e = int(np.flatnonzero(t[:, 6] != 0xFF)[-1])
        word, n = int(t[e, :4].copy().view(np.uint32)[0]), BLOCK * BLOCK
        values = _unpack(self.payload[word:], t[e, 6], n)
        first = self.payload.size - 2
        self.payload = np.concatenate([self.payload[:-2], np.array(pack_plain(values, 13) + [0, 0], np.uint32)])
        t[e, :4] = np.array([first], np.uint32).view(np.uint8)
        t[e, 6] = 13

    def widen_vectors(self, c, l, change=None):
        """The vectors of (channel, level) again, in a 13-bit sequence;
        change(values): (mx + 4W, my + 4W) of every record, in place."""
        d = self.head[176 + (c * 8 + l) * 16:][:16]
        word, count = int(d[:4].copy().view(np.uint32)[0]), int(d[8:12].copy().view(np.uint32)[0])
        values = _unpack(self.mv[word:], d[12], 2 * count)
        if change:
            change(values)
        first = self.mv.size - 2
        self.mv = np.concatenate([self.mv[:-2], np.array(pack_plain(values, 13) + [0, 0], np.uint32)])
        d[:4] = np.array([first], np.uint32).view(np.uint8)
        d[12] = 13


def _far(values):
    values[::7] = 4000  # quarter pixels, less the window's bias: beyond 12 signed bits


def _variants():
    s = _Stream(_base())
    yield "as encoded", s.build(), True
    s.widen_block()
    yield "wide block", s.build(), True
    s = _Stream(_base())
    for c in range(3):
        s.widen_vectors(c, 0)
    yield "wide vectors", s.build(), True
    for c in (0, 2):
        s = _Stream(_base())
        s.widen_vectors(c, 0, _far)
        yield "far vectors of channel %d" % c, s.build(), False
    for c, add in ((0, 9000), (1, -9000)):
        s = _Stream(_base())
        root = s.root.view(np.int16)
        full = root.size * 2 // 3  # luma, then two channels of a quarter each
        part = root[:full] if c == 0 else root[full:full + full // 4]
        part[::3] += add
        yield "values of channel %d beyond the lanes" % c, s.build(), False


VARIANTS = ("as encoded", "wide block", "wide vectors", "far vectors of channel 0", "far vectors of channel 2",
            "values of channel 0 beyond the lanes", "values of channel 1 beyond the lanes")


@pytest.mark.parametrize("name", VARIANTS)
def test_pixels(name):
    import torch

    from paper_1902_09396_amd import lf

    stream = next(s for n, s, _ in _variants() if n == name)
    o, field = oracle.OracleLF(stream), lf.LightField(stream)
    cams = np.concatenate([lfscene.random_pinhole_cameras(3, 8, 8, 64, 64, 45, 50, seed=2),
                           lfscene.camera_path_orbit(3, 8, 8, 64, 64, 45, 50, radius=2.0)])
    dc = torch.from_numpy(cams).cuda()
    got = field.render_views(dc, 45, 50)
    assert torch.equal(got, field.render_views(dc, 45, 50, per_ray=True))
    assert np.abs(got.cpu().numpy() - o.render(cams, 45, 50)).max() <= 1e-5
    for level in range(LEVELS + 1):
        lod = field.render_views_lod(level, dc, 45, 50).cpu().numpy()
        assert np.abs(lod - o.render_lod(level, cams, 45, 50)).max() <= 1e-5, level


@pytest.mark.parametrize("name", VARIANTS[1:3])
def test_values_in_range_keep_the_tiles(name):
    """The same values in wider sequences cost the same (ten times that one
    thread per ray)."""
    import torch

    from paper_1902_09396_amd import lf

    streams = {n: s for n, s, _ in _variants()}
    dc = torch.from_numpy(lfscene.random_pinhole_cameras(8, 8, 8, 64, 64, WO, HO, seed=4)).cuda()
    times, images = [], []
    for n in ("as encoded", name):
        field = lf.LightField(streams[n])
        images.append(field.render_views(dc, WO, HO))
        best = float("inf")
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                field.render_views(dc, WO, HO)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        times.append(best)
    assert torch.equal(*images)
    assert times[1] < 2 * times[0], times
