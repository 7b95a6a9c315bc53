"""The bins of the tile kernel's GELU output (host code, no GPU): which scales have them, and that a value's code by bin
is the oracle's around every step and over the whole line."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from test_gelu_breakpoints import _neighbours

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# the kernel's lookup on the host: the bin by one fma, clamped and truncated, then one comparison
LOOKUP = r"""
#include <cmath>
#include <cstring>
#include "rmsmp_internal.h"
extern "C" int codes_by_bin(float inv_s, int z, const float* y, long n, unsigned char* out, float* steps) {
  rmsmp::GeluTable t;
  rmsmp::GeluBins b;
  rmsmp::gelu_table(inv_s, z, &t);
  rmsmp::gelu_bins(t, &b);
  constexpr int BINS = rmsmp::GeluBins::BINS;
  float step[BINS];
  unsigned char below[BINS], from[BINS];
  for (int i = 0; i < BINS; ++i) {
    step[i] = INFINITY, below[i] = from[i] = b.code[0];
    for (int k = 0; k < b.n; ++k) {
      const int bin = (int)std::fmaf(b.step[k], b.scale, b.offset);
      if (bin == i) step[i] = b.step[k], from[i] = b.code[k + 1];
      if (bin < i) below[i] = from[i] = b.code[k + 1];
    }
  }
  for (long i = 0; b.n && i < n; ++i) {
    const int bin = (int)std::fmin(std::fmax(std::fmaf(y[i], b.scale, b.offset), 0.0f), (float)(BINS - 1));
    out[i] = y[i] >= step[bin] ? from[bin] : below[bin];
  }
  std::memcpy(steps, b.step, sizeof(b.step));
  return b.n;
}
"""


@pytest.fixture(scope="module")
def codes_by_bin(tmp_path_factory):
    d = tmp_path_factory.mktemp("bins")
    csrc = os.path.join(ROOT, "paper_2111_00153_amd", "csrc")
    (d / "lookup.cpp").write_text(LOOKUP)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I" + csrc, "-I" + os.path.join(ROOT, "include"), str(d / "lookup.cpp"),
                           os.path.join(csrc, "gelu_host.cpp"), "-o", str(d / "lookup.so")])
    f = ctypes.CDLL(str(d / "lookup.so")).codes_by_bin
    f.argtypes = [ctypes.c_float, ctypes.c_int, ctypes.c_void_p, ctypes.c_long, ctypes.c_void_p, ctypes.c_void_p]

    def call(inv_s, z, y):
        out, steps = np.full(y.size, 255, np.uint8), np.empty(31, np.float32)
        n = f(inv_s, z, y.ctypes.data, y.size, out.ctypes.data, steps.ctypes.data)
        return n, out, steps[:n]
    return call


# (the scales of the GPU test of the same codes: both ways of the kernel are in it)
# No bins: steps a scale apart around 0 beside steps far out on the falling branch, which 64 equal bins do not separate.
@pytest.mark.parametrize("s_out,z_out,binned", [(0.18, 1, True), (0.18, 15, True), (0.05, 4, True), (1.0, 0, True), (40.0, 3, True),
                                                (0.011, 14, False), (1e-3, 7, False), (1e-4, 15, False)])
def test_codes_by_bin_are_the_oracles(oracle, codes_by_bin, s_out, z_out, binned):
    inv = float(np.float32(1.0 / s_out))
    n, _, steps = codes_by_bin(inv, z_out, np.zeros(1, np.float32))
    assert (n > 0) == binned
    if not n:
        return
    rng = np.random.default_rng(z_out)
    y = np.concatenate([_neighbours(s) for s in steps] +
                       [np.linspace(-12.0, 24.0, 100001, dtype=np.float32), np.float32([-3e38, -1e10, 1e10, 3e38, 0.0, -0.0]),
                        (rng.standard_normal(100000) * rng.choice([0.01, 0.3, 1.0, 4.0, 30.0], 100000)).astype(np.float32)])
    _, out, _ = codes_by_bin(inv, z_out, y)
    assert np.array_equal(out, oracle.gelu_codes(y, inv, z_out)[1])
