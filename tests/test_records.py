"""The slice records of the kernels, compiled for the CPU: what is packed into self-validating words comes out again
bit for bit (csrc/records.h holds bit arithmetic only, so the kernels and this test run the same source)."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "records.h"
using namespace adasd;
extern "C" void draw(int n, const float* f, const int* i1, const unsigned char* poison, uint64_t* words, float* f_out,
                     int* i1_out, unsigned char* poison_out) {
  for (int k = 0; k < n; ++k) {
    uint64_t w[3];
    pack_draw(DrawRecord{f[4 * k], f[4 * k + 1], f[4 * k + 2], f[4 * k + 3], i1[k], poison[k] != 0}, w);
    for (int j = 0; j < 3; ++j) words[3 * k + j] = w[j];
    const DrawRecord r = unpack_draw(w);
    f_out[4 * k] = r.k1; f_out[4 * k + 1] = r.k2; f_out[4 * k + 2] = r.zp; f_out[4 * k + 3] = r.zq;
    i1_out[k] = r.i1;
    poison_out[k] = r.poison;
  }
}
extern "C" void draft(int n, const float* f, const int* i1, uint64_t* words, float* f_out, int* i1_out) {
  for (int k = 0; k < n; ++k) {
    uint64_t w[3];
    pack_draft(DraftRecord{f[5 * k], f[5 * k + 1], f[5 * k + 2], f[5 * k + 3], f[5 * k + 4], i1[k]}, w);
    for (int j = 0; j < 3; ++j) words[3 * k + j] = w[j];
    const DraftRecord r = unpack_draft(w);
    f_out[5 * k] = r.m; f_out[5 * k + 1] = r.s; f_out[5 * k + 2] = r.u; f_out[5 * k + 3] = r.k1; f_out[5 * k + 4] = r.k2;
    i1_out[k] = r.i1;
  }
}
extern "C" void pair(int n, const float* f, uint64_t* words, float* f_out) {
  for (int k = 0; k < n; ++k) {
    uint64_t w[3];
    const float* x = f + 6 * k;
    pack_pair(PairRecord{x[0], x[1], x[2], x[3], x[4], x[5]}, w);
    for (int j = 0; j < 3; ++j) words[3 * k + j] = w[j];
    const PairRecord r = unpack_pair(w);
    const float y[6] = {r.mp, r.sp, r.up, r.mq, r.sq, r.uq};
    for (int j = 0; j < 6; ++j) f_out[6 * k + j] = y[j];
  }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("records")
    (d / "records.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2512_11280_amd", "csrc"),
                    str(d / "records.cpp"), "-o", str(d / "records.so")], check=True)
    return C.CDLL(str(d / "records.so"))


def _floats(n, seed):
    """Any bit pattern: both values of the lowest bit, zeros, infinities, the type's ends, NaN."""
    x = np.random.default_rng(seed).integers(0, 1 << 32, n, dtype=np.uint64).astype(np.uint32)
    edges = np.array([0.0, -0.0, np.inf, -np.inf, 3.4028235e38, -3.4028235e38, 1e-45, 1.0, -1.0, 300.0], np.float32)
    x[:edges.size] = edges.view(np.uint32)
    return x.view(np.float32)


def _p(a):
    return a.ctypes.data_as(C.c_void_p)


def test_draw_records_arrive_as_they_were_sent(lib):
    n = 20000
    f = np.stack([_floats(n, s) for s in range(4)], 1).copy()
    rng = np.random.default_rng(9)
    i1 = rng.integers(-1, 1 << 24, n).astype(np.int32)
    i1[:2] = -1, (1 << 24) - 1
    poison = rng.integers(0, 2, n).astype(np.uint8)
    words, f2, i2, p2 = np.zeros((n, 3), np.uint64), np.zeros_like(f), np.zeros_like(i1), np.zeros_like(poison)
    lib.draw(n, _p(f), _p(i1), _p(poison), _p(words), _p(f2), _p(i2), _p(p2))
    assert (words & np.uint64(1)).all()                       # every word says that it is there
    assert np.array_equal(f.view(np.uint32), f2.view(np.uint32))
    assert np.array_equal(i1, i2) and np.array_equal(poison, p2)


def test_draft_records_arrive_as_they_were_sent(lib):
    n = 20000
    f = np.stack([_floats(n, 20 + s) for s in range(5)], 1).copy()
    f[:, 0] = (f[:, 0].view(np.uint32) | 1).view(np.float32)          # a reference carries the flag
    f[:, 1] = np.abs(f[:, 1])                                         # a sum of exponentials has no sign
    i1 = np.random.default_rng(29).integers(-1, 1 << 24, n).astype(np.int32)
    words, f2, i2 = np.zeros((n, 3), np.uint64), np.zeros_like(f), np.zeros_like(i1)
    lib.draft(n, _p(f), _p(i1), _p(words), _p(f2), _p(i2))
    assert (words & np.uint64(1)).all()
    assert np.array_equal(f.view(np.uint32), f2.view(np.uint32)) and np.array_equal(i1, i2)


def test_row_pair_records_arrive_as_they_were_sent(lib):
    n = 20000
    f = np.stack([_floats(n, 40 + s) for s in range(6)], 1).copy()
    for c in (0, 3):
        f[:, c] = (f[:, c].view(np.uint32) | 1).view(np.float32)
    for c in (1, 4):
        f[:, c] = np.abs(f[:, c])
    words, f2 = np.zeros((n, 3), np.uint64), np.zeros_like(f)
    lib.pair(n, _p(f), _p(words), _p(f2))
    assert (words & np.uint64(1)).all()
    assert np.array_equal(f.view(np.uint32), f2.view(np.uint32))
