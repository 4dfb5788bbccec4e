"""Host allocation failure inside the library's calls: a status or the work
done on the calling thread, never a C++ exception out of a C entry point."""

import os
import subprocess
import sys

import numpy as np

from conftest import ROOT, stream_for

SHIM = """
#include <cstdlib>
#include <new>
static volatile int fail;
extern "C" void set_fail(int on) { fail = on; }
void* operator new(std::size_t n)
{
    void* p = fail ? nullptr : std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }
"""

CALL = """
import ctypes as C, sys
shim = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)  # before every user of operator new
import numpy as np
from paper_1902_09396_amd import lf
s = np.load(sys.argv[2])
need = C.c_int64()
lib = lf.lib()
shim.set_fail(1)
status = lib.lf_query_arena(s.ctypes.data, s.size, C.byref(need))
shim.set_fail(0)
print(status, need.value, lf.query_arena(s))
"""


def test_table_scan_without_memory(tmp_path, tiny_lf):
    """A table large enough for several threads, none of which can start."""
    (tmp_path / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", str(tmp_path / "shim.so"), str(tmp_path / "shim.cpp")], check=True)
    np.save(tmp_path / "stream.npy", stream_for("tiny", tiny_lf, block=2))
    r = subprocess.run([sys.executable, "-c", CALL, str(tmp_path / "shim.so"), str(tmp_path / "stream.npy")], cwd=ROOT,
                       capture_output=True, text=True, timeout=300, env=dict(os.environ, PYTHONPATH=ROOT))
    assert r.returncode == 0, r.stderr[-2000:]
    status, got, expect = (int(v) for v in r.stdout.split()[-3:])
    assert status == 0 and got == expect
