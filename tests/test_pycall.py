"""The native marshalling module: what it hands over, what it refuses, and how it leaves.  CPU only: the functions it
calls are replaced by ones that record their arguments."""
import ctypes
import subprocess
import sys
import os

import pytest

torch = pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

THROWS = r"""
#include <stdexcept>
extern "C" int throws_standard(...) { throw std::runtime_error("from inside the call"); }
extern "C" int throws_other(...) { throw 7; }
"""

RAISES = r"""
import ctypes, sys, threading
import torch
import paper_2111_00153_amd as rm
from paper_2111_00153_amd import _pycall
lib = ctypes.CDLL(sys.argv[1])
for name, text in (("throws_standard", "from inside the call"), ("throws_other", "unknown")):
    _pycall.bind(*[ctypes.cast(getattr(lib, name), ctypes.c_void_p).value] * 4)
    for _ in range(3):
        try:
            _pycall.gemm(None, None, 1, rm.make_epilogue(), None, 0)
        except RuntimeError as e:
            assert text in str(e), e
        else:
            raise SystemExit("no exception")
    # the interpreter's lock is held again: other threads run and are waited for
    t = threading.Thread(target=lambda: None)
    t.start()
    t.join()
print("left in order")
"""


def test_a_call_that_throws_takes_the_interpreters_lock_back(tmp_path):
    """In a process of its own: raised without the lock, the exception ends the interpreter."""
    src, lib = tmp_path / "throws.cpp", tmp_path / "throws.so"
    src.write_text(THROWS)
    subprocess.check_call(["g++", "-shared", "-fPIC", "-o", str(lib), str(src)])
    r = subprocess.run([sys.executable, "-c", RAISES, str(lib)], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "left in order" in r.stdout, (r.returncode, r.stdout, r.stderr[-2000:])
