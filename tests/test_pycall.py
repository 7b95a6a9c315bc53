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


class Stand:
    """Stands for a GPU tensor: the attributes the module asks a tensor of another type for."""

    def __init__(self, address, shape=(3, 4), cuda=True, contiguous=True):
        self.address, self.shape, self.is_cuda, self.contiguous = address, shape, cuda, contiguous

    def is_contiguous(self):
        return self.contiguous

    def data_ptr(self):
        return self.address


class StandStream:
    cuda_stream = 0x5000


class Subclass(torch.Tensor):
    """A tensor type of its own: what it says of itself counts."""
    is_cuda = True


@pytest.fixture
def recorded():
    """The module with functions that record their arguments in the place of the library's; -> (binding, module, list)."""
    import paper_2111_00153_amd as rm
    from paper_2111_00153_amd import _pycall, binding
    P, I64, SZ, calls = ctypes.c_void_p, ctypes.c_int64, ctypes.c_size_t, []

    def recorder(name, *types):
        def record(*a):
            calls.append((name, tuple(v or 0 for v in a)))
            return 0
        return ctypes.CFUNCTYPE(ctypes.c_int, *types)(record)
    fakes = [recorder("gemm", P, P, I64, P, P, P), recorder("conv2d", P, P, P, P, P, P, SZ, P),
             recorder("fake_quant_rows", P, I64, I64, P, P, P, P, P), recorder("ste_backward", P, P, P, I64, I64, P, P)]
    _pycall.bind(*[ctypes.cast(f, P).value for f in fakes])
    yield rm, _pycall, calls
    _pycall.bind(*(ctypes.cast(getattr(binding._lib, n), P).value for n in ("rmsmp_gemm", "rmsmp_conv2d", "rmsmp_fake_quant_rows", "rmsmp_ste_backward")))


def test_arguments_arrive(recorded):
    rm, m, calls = recorded
    ep, d, h = rm.make_epilogue(), rm.ConvDesc(1, 2, 3, 4, 1, 1, 1, 0), ctypes.c_void_p(0x100)
    ea, da = ctypes.addressof(ep), ctypes.addressof(d)
    X, Y, Z, S = Stand(0x1000), Stand(0x2000), Stand(0x3000), Stand(0x4000)
    assert m.gemm(h, X, 1 << 40, ep, Y, StandStream()) == 0
    assert m.gemm(None, None, -1, ep, None, 7) == 0
    assert m.conv2d(h, X, d, ep, Y, Z, 96, 0) == 0
    assert m.conv2d(h, X, d, ep, Y, None, 0, StandStream()) == 0
    assert m.fake_quant_rows(X, S, Y, None, Z, 7) == 0
    assert m.ste_backward(X, Y, None, None, 7) == 0
    assert m.ste_backward(X, Y, Z, S, StandStream()) == 0
    assert calls == [("gemm", (0x100, 0x1000, 1 << 40, ea, 0x2000, 0x5000)), ("gemm", (0, 0, -1, ea, 0, 7)),
                     ("conv2d", (0x100, 0x1000, da, ea, 0x2000, 0x3000, 96, 0)), ("conv2d", (0x100, 0x1000, da, ea, 0x2000, 0, 0, 0x5000)),
                     ("fake_quant_rows", (0x1000, 3, 4, 0x4000, 0, 0x2000, 0x3000, 7)),
                     ("ste_backward", (0, 0, 0x1000, 3, 4, 0x2000, 7)), ("ste_backward", (0x3000, 0x4000, 0x1000, 3, 4, 0x2000, 0x5000))]


def test_a_tensor_subclass_is_asked_for_what_it_says_of_itself(recorded):
    rm, m, calls = recorded
    t = torch.zeros(3, 4).as_subclass(Subclass)
    m.gemm(None, t, 1, rm.make_epilogue(), None, 0)
    assert calls[0][1][1] == torch.Tensor.data_ptr(t)
    with pytest.raises(ValueError):
        m.gemm(None, torch.zeros(4, 3).t().as_subclass(Subclass), 1, rm.make_epilogue(), None, 0)
    assert len(calls) == 1


class WatchingMode(torch.overrides.TorchFunctionMode):
    def __torch_function__(self, func, types, args=(), kwargs=None):
        if getattr(func, "__name__", "") == "__get__" and getattr(func.__self__, "__name__", "") == "is_cuda":
            return True
        return func(*args, **(kwargs or {}))


def test_a_function_mode_sees_the_questions(recorded):
    rm, m, calls = recorded
    t, ep = torch.zeros(3, 4), rm.make_epilogue()
    with WatchingMode():
        m.gemm(None, t, 1, ep, None, 0)
    assert calls[0][1][1] == t.data_ptr()


def test_what_is_refused_never_reaches_the_library(recorded):
    rm, m, calls = recorded
    ep, d, X, h = rm.make_epilogue(), rm.ConvDesc(1, 2, 3, 4, 1, 1, 1, 0), Stand(0x1000), ctypes.c_void_p(0x100)
    other = ctypes.c_int32(0)
    for bad in (torch.zeros(3, 4), Stand(0, cuda=False), Stand(0, contiguous=False)):
        for call in (lambda: m.gemm(h, bad, 1, ep, X, 0), lambda: m.gemm(h, X, 1, ep, bad, 0), lambda: m.conv2d(h, X, d, ep, X, bad, 0, 0),
                     lambda: m.fake_quant_rows(X, bad, X, None, None, 0), lambda: m.fake_quant_rows(X, X, X, bad, None, 0),
                     lambda: m.ste_backward(X, bad, None, None, 0), lambda: m.ste_backward(X, X, bad, X, 0)):
            with pytest.raises(ValueError):
                call()
    for call in (lambda: m.gemm(h, X, 1, other, X, 0), lambda: m.gemm(h, X, 1, d, X, 0), lambda: m.gemm(h, X, 1, None, X, 0), lambda: m.gemm(other, X, 1, ep, X, 0),
                 lambda: m.gemm(7, X, 1, ep, X, 0), lambda: m.gemm(h, X, 1.5, ep, X, 0), lambda: m.gemm(h, X, 1, ep, X), lambda: m.conv2d(h, X, ep, ep, X, None, 0, 0),
                 lambda: m.gemm(h, X, 1, ep, X, [])):
        with pytest.raises(TypeError):
            call()
    with pytest.raises(AttributeError):
        m.gemm(h, object(), 1, ep, X, 0)
    with pytest.raises(ValueError):
        m.ste_backward(Stand(0x1000, shape=(3, 4, 5)), X, None, None, 0)
    assert calls == []


def test_a_freed_layer_is_refused_by_the_library():
    import paper_2111_00153_amd as rm

    class Freed:
        handle = None
    with pytest.raises(rm.RmsmpError) as e:
        rm.rmsmp_gemm(Freed, None, 1, rm.make_epilogue(), None, 0)
    assert e.value.code == 1


@pytest.mark.gpu
def test_tensor_types_and_streams_on_the_gpu():
    """A plain tensor, a subclass, a function mode; torch's current stream, a stream object, its number: one result."""
    import numpy as np
    import paper_2111_00153_amd as rm
    import synth_inputs as si
    rng = np.random.default_rng(4)
    M, K, N = 34, 96, 20
    p = rm.rmsmp_pack_weights(si.weights_rowscaled(rng, M, K), si.scheme_permutation(rng, rm.rmsmp_ratio_counts(M, 35, 60, 5)))
    X = torch.from_numpy(rm.pack_u4(si.act_codes_u4(rng, (N, K)))).to("cuda:0")
    ep = rm.make_epilogue(0.05, 0, 4, None, False, rm.OUT_INT32)
    want = torch.empty((M, N), dtype=torch.int32, device="cuda:0")
    rm.rmsmp_gemm(p, X, N, ep, want)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()

    class Plain(torch.Tensor):
        pass

    for x, stream in ((X, side), (X, side.cuda_stream), (X.as_subclass(Plain), None), (X.as_subclass(Plain), side)):
        Y = torch.full_like(want, -777)
        torch.cuda.synchronize()
        rm.rmsmp_gemm(p, x, N, ep, Y, stream)
        torch.cuda.synchronize()
        assert torch.equal(Y, want)
    Y = torch.full_like(want, -777)
    with torch.overrides.BaseTorchFunctionMode():
        rm.rmsmp_gemm(p, X, N, ep, Y)
    torch.cuda.synchronize()
    assert torch.equal(Y, want)
    p.free()
