"""The arithmetic of the noise that the kernels share (csrc/noise_series.h).  Error of log2 E, E = -ln u of a 32-bit noise word, as the scans form it, against 64 bits: the kernels' own series
(csrc/noise_series.h) compiled for the CPU, with logarithms that are exact to a rounding.  The bound is what five Taylor
terms below t = 1/16 reach (largest error 1.11e-6, which is the rounding of values near -32; 1.29e-7 rms)."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cmath>
#include "noise_series.h"
using namespace adasd;
static float lg2(float x) { return (float)std::log2((double)x); }
extern "C" void errors(long n, const uint32_t* words, double* largest, double* rms) {
  double worst = 0, sum = 0;
  for (long k = 0; k < n; ++k) {
    const uint32_t w = words[k];
    const float u = __builtin_fmaf((float)w, 0x1p-32f, 0x1p-33f), t = __builtin_fmaf((float)(~w), 0x1p-32f, 0x1p-33f);
    const float lE = lg2(std::fabs(t < kSerBelow ? log2_series(t) : lg2(u)));   // log2 of -log2 u
    const double td = ((double)(~w) + 0.5) * 0x1p-32, ud = ((double)w + 0.5) * 0x1p-32;
    const double exact = std::log2(-(td < 0.5 ? std::log1p(-td) : std::log(ud)) / 0.69314718055994530942);
    const double e = std::fabs((double)lE - exact);
    if (e > worst) worst = e;
    sum += e * e;
  }
  *largest = worst;
  *rms = std::sqrt(sum / n);
}
// Largest (key - floor) of the elements that would be left out: words[k] with the keys without noise at which the bound comes
// closest, times below[k], and the three floats that follow.
extern "C" void bounds(long n, const uint32_t* words, const double* below, double* largest, long* left_out) {
  *largest = -INFINITY;
  *left_out = 0;
  for (long k = 0; k < n; ++k) {
    const uint32_t w = words[k];
    const double td = ((double)(~w) + 0.5) * 0x1p-32, ud = ((double)w + 0.5) * 0x1p-32;
    const double E2 = -(td < 0.5 ? std::log1p(-td) : std::log(ud)) / 0.69314718055994530942;     // -log2 u
    float ef = (float)((4294967296.0 - (double)w) * below[k]);
    for (int step = 0; step < 4; ++step, ef = std::nextafterf(ef, INFINITY)) {
      if (!(noise_reach(ef, 1.0f, w) <= kNoiseTop)) continue;
      const double over = std::log2((double)ef) - (double)kReach - std::log2(E2);                 // key - floor
      if (over > *largest) *largest = over;
      ++*left_out;
    }
  }
}
// Flat rows of logit z: keys as the scans form them, words[k] seen first and others[k] after it.  How many of the others are left
// out, and how many of those should not have been (within the guard of the first key, or above it).
extern "C" void large(long n, float z, const uint32_t* words, const uint32_t* others, long* left_out, long* wrong) {
  const float log2e = 1.44269504088896340736f;
  auto key = [&](uint32_t w) {
    const double td = ((double)(~w) + 0.5) * 0x1p-32, ud = ((double)w + 0.5) * 0x1p-32;
    const float lE = (float)std::log2(-(td < 0.5 ? std::log1p(-td) : std::log(ud)) / 0.69314718055994530942);
    return __builtin_fmaf(z, log2e, -lE);
  };
  *left_out = *wrong = 0;
  for (long k = 0; k < n; ++k) {
    const float first = key(words[k]), lift = -floor_of(first);
    const float e = (float)std::exp2((double)__builtin_fmaf(z, log2e, lift));
    if (!(noise_reach(e, 1.0f, others[k]) <= kNoiseTop)) continue;
    ++*left_out;
    *wrong += !((double)first - (double)key(others[k]) > 0x1p-13);
  }
}
// While nothing has been looked at: may an element win, by its logit (the lift of a row's logits) or by its weight e (the factor)?
extern "C" int first_by_logit(float z, uint32_t word) {
  const float t = __builtin_fmaf(z, 1.44269504088896340736f, -kNoFloor);
  return !(noise_reach((float)std::exp2((double)t), 1.0f, word) <= kNoiseTop);
}
extern "C" int first_by_weight(float e, uint32_t word) {
  return !(noise_reach(e, (float)std::exp2((double)reach_exponent(-kNoFloor)), word) <= kNoiseTop);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("noise")
    (d / "noise.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2512_11280_amd", "csrc"), str(d / "noise.cpp"), "-o", str(d / "noise.so")], check=True)
    return C.CDLL(str(d / "noise.so"))


def _errors(lib, words):
    words = np.ascontiguousarray(words, np.uint32)
    largest, rms = C.c_double(), C.c_double()
    lib.errors(C.c_long(words.size), words.ctypes.data_as(C.c_void_p), C.byref(largest), C.byref(rms))
    return largest.value, rms.value


@pytest.mark.parametrize("lo,hi", [(0, 1 << 32), (0, 4096), ((1 << 32) - 65536, 1 << 32), (1 << 31, (1 << 31) + 4096),
                                   ((1 << 32) - (1 << 23), (1 << 32) - (1 << 21))])
def test_what_is_left_out_cannot_win(lib, lo, hi):
    """Whatever the word and the logit: an element that the scans leave out has its key below the floor by the guard
    (2^-13) at least."""
    rng = np.random.default_rng(lo % 997)
    words = rng.integers(lo, hi, 400_000, dtype=np.uint64).astype(np.uint32)
    words[:4] = [lo, hi - 1, lo, hi - 1]
    below = np.where(rng.random(words.size) < 0.5, 1.0, np.exp2(-rng.uniform(0, 40, words.size)))
    below[rng.random(words.size) < 0.2] = 1.0 - 2.0**-20
    largest, left = C.c_double(), C.c_long()
    lib.bounds(C.c_long(words.size), words.ctypes.data_as(C.c_void_p), below.ctypes.data_as(C.c_void_p), C.byref(largest), C.byref(left))
    print(f"left out {left.value}, largest key over the floor {largest.value:.3e}")
    assert left.value > 1000 and largest.value < -2.0**-13


@pytest.mark.parametrize("z", [0.0, 30.0, 700.0, -5000.0, 65536.0, 1.0e6, -1.0e7, 1.0e7, 3.0e8])
def test_what_is_left_out_cannot_win_among_large_logits(lib, z):
    """Large logits have keys whose own roundings outgrow the guard.  Noise words near the top, whose keys lead a row, against
    words a little below: by so much that the other key is a rounding or two lower."""
    rng = np.random.default_rng(5)
    E = 10.0 ** rng.uniform(-7, -1, 400_000)              # -ln u of the first, and of the other one
    ulp = np.spacing(np.float32(abs(z) * 1.4427 + 30))
    other = E * np.exp2(rng.uniform(0, 1, E.size) ** 2 * 4 * max(ulp, 1e-2))
    words, others = ((np.exp(-x) * 2.0**32).clip(0, 2.0**32 - 1).astype(np.uint32) for x in (E, other))
    left, wrong = C.c_long(), C.c_long()
    lib.large(C.c_long(words.size), C.c_float(z), words.ctypes.data_as(C.c_void_p), others.ctypes.data_as(C.c_void_p),
              C.byref(left), C.byref(wrong))
    print(f"z = {z}: left out {left.value}, wrongly {wrong.value}")
    assert wrong.value == 0 and (left.value > 1000 or z > 1e8)


@pytest.mark.parametrize("word", [0, 1 << 31, (1 << 32) - 4096])
def test_masked_logits_fall_out_before_anything_has_been_looked_at(lib, word):
    by_logit = lambda z: lib.first_by_logit(C.c_float(z), C.c_uint32(word))
    by_weight = lambda e: lib.first_by_weight(C.c_float(e), C.c_uint32(word))
    assert not by_logit(-np.inf) and not by_weight(0.0)
    assert all(by_logit(z) for z in (-2e38, -1e30, -1e4, 0.0, 50.0, 1e38, np.inf, np.nan))
    assert all(by_weight(e) for e in (2.0**-94, 2.0**-38, 1.0, 2.0**20, np.inf, np.nan))


def test_error_over_the_whole_range(lib):
    largest, rms = _errors(lib, np.random.default_rng(0).integers(0, 1 << 32, 4_000_000, dtype=np.uint64))
    print(f"log2 E: largest error {largest:.3e}, rms {rms:.3e}")
    assert largest < 1.11e-6 and rms < 1.29e-7


@pytest.mark.parametrize("lo,hi", [(0, 1 << 20), (1 << 31, (1 << 31) + (1 << 20)), ((1 << 32) - (1 << 20), 1 << 32),
                                   (int((1 - 1 / 11) * 2**32), int((1 - 1 / 13) * 2**32)),
                                   (int((1 - 1 / 15) * 2**32), int((1 - 1 / 17) * 2**32)),
                                   (int((1 - 1 / 60) * 2**32), int((1 - 1 / 68) * 2**32))])
def test_error_where_it_can_be_largest(lib, lo, hi):
    """The ends of the range, and both sides of every line the series has been cut at."""
    words = lo + np.arange(0, hi - lo, max(1, (hi - lo) >> 20), dtype=np.uint64)
    assert _errors(lib, words)[0] < 1.11e-6
