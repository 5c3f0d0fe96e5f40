"""A batch call without a request array is refused before anything is sized by
its count."""

import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CODE = """
import ctypes, resource
from paper_2304_08159_amd import _lib
lib = _lib.load()
res = (_lib.BatchResult if "poisson" in {name!r} else _lib.NsResult)()
before = resource.getrusage(resource.RUSAGE_SELF).ru_maxrss
st = lib.{name}(None, 2 ** 31 - 1, ctypes.c_void_p(256), 1 << 40, None, ctypes.byref(res))
grown = (resource.getrusage(resource.RUSAGE_SELF).ru_maxrss - before) >> 10
assert st == _lib.WL_ERR_INVALID_ARG and b"NULL" in lib.wl_last_error(), st
assert grown < 256, grown
"""


@pytest.mark.parametrize("name", ["wl_poisson_batch_solve", "wl_ns_batch_run"])
def test_null_requests_are_refused(name):
    from paper_2304_08159_amd import _lib
    if not os.path.exists(_lib.LIB_PATH):
        pytest.skip("libwl.so not built")
    r = subprocess.run([sys.executable, "-c", CODE.format(name=name)], cwd=ROOT,
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
