"""Host checks of a block table large enough to be scanned by several threads."""

import numpy as np
import pytest

from conftest import stream_for


@pytest.fixture(scope="module")
def stream(tiny_lf):
    return stream_for("tiny", tiny_lf, block=2)  # 245,760 entries


def _table(s):
    off, size = s[128:144].copy().view(np.uint64)
    assert size // 8 > 1 << 16
    return int(off), int(size) // 8


@pytest.mark.parametrize("byte,value,word", [(6, 0x7F, "mode"), (3, 0xFF, "payload"), (6, 20, "range")])
def test_first_bad_entry_is_reported(stream, byte, value, word):
    from paper_1902_09396_amd import lf

    lf.query_arena(stream)  # sound as it is
    off, n = _table(stream)
    significant = np.flatnonzero(stream[off + 6:off + 8 * n:8] != 0xFF)
    for picks in ((0,), (-1,), (len(significant) // 3, len(significant) // 2), (5, -2)):
        bad = stream.copy()
        for k in picks:
            e = significant[k]
            bad[off + 8 * e + byte] = value
            if word == "range":  # 21-bit quint values times the step
                bad[off + 8 * e + 6] = (2 << 5) | 20
                bad[off + 8 * e:off + 8 * e + 4] = 0
        first = min(int(significant[k]) for k in picks)
        if word == "range":
            bad = bad.copy()
            bad[48:80].view(np.int32)[:] = 4096
        with pytest.raises(lf.LFError) as err:
            lf.query_arena(bad)
        assert err.value.status == lf.LF_EFORMAT and word in str(err.value)
        if word == "mode":
            assert "entry %d" % first in str(err.value)
