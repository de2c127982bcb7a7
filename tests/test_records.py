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
extern "C" int last(int before, int S) { return last_to_add(before, S); }
extern "C" int come(int before, int added) { return last_to_come(before, added); }
extern "C" int undecided(uint64_t set) { return deciding(set); }
extern "C" int missing(uint64_t set, int s) { return is_missing(set, s); }
extern "C" uint64_t mark() { return kDeciding; }
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


@pytest.mark.parametrize("few", [False, True])
@pytest.mark.parametrize("S", [2, 3, 4])
def test_every_row_is_folded_once_and_leaves_no_word_behind(lib, few, S):
    """All orders in which the slices of a row can send, their words and additions can take effect, and the last slice of few rows
    can give up, also before the others have started: one of them folds, after all have sent and with all words there, and
    words, count and set are zero at the end, so that the next call finds nothing of this one.  (A record of two words here.)"""
    lib.mark.restype = C.c_uint64
    mark, undecided, missing = lib.mark(), lambda v: lib.undecided(C.c_uint64(v)), lambda v, s: lib.missing(C.c_uint64(v), s)
    assert undecided(mark) and not undecided((1 << 63) - 1) and missing(1 << 62, 62) and not missing(1 << 62, 61)
    last, none, names = S - 1, ((False, False),) * S, ("there", "sent", "at", "count", "set_", "left", "found", "folds")
    # of each slice: its words that are there, its words that have got there, what it does next.  Then: count, set, and of the last
    # slice: those it still has to look at, those it found missing.  How often the row was folded.
    start = (none, none, ("start",) * S, 0, 0, frozenset(), frozenset(), 0)
    seen, todo, ends = {start}, [start], 0

    def put(t, s, v):
        return t[:s] + (v,) + t[s + 1:]
    while todo:
        state = todo.pop()
        there, sent, at, count, set_, left, found, folds = state
        new = []

        def go(**kw):
            new.append(tuple(kw.get(n, v) for n, v in zip(names, state)))

        def add(s, n, mine):                              # (the last to come clears the set)
            go(count=count + n, set_=0 if mine else set_, at=put(at, s, "folds" if mine else "done"))
        for s in range(S):
            if at[s] == "start":
                go(at=put(at, s, "adds" if not few else "reads" if s == last else "waits"))
                continue
            for i in range(2):
                if not sent[s][i]:
                    go(there=put(there, s, put(there[s], i, True)), sent=put(sent, s, put(sent[s], i, True)))
            if at[s] == "adds":
                mine = lib.last(count, S)
                go(count=0 if mine else count + 1, at=put(at, s, "folds" if mine else "done"))
            if at[s] == "waits" and all(sent[s]):         # its record has got there: it looks at the set
                go(at=put(at, s, "done" if set_ == 0 else "looks"))
            if at[s] == "looks" and not undecided(set_):
                go(at=put(at, s, "comes" if missing(set_, s) else "done"))
            if at[s] == "comes":
                add(s, 1, lib.come(count, 1))
            if at[s] == "reads":
                if all(map(all, there)):
                    go(at=put(at, s, "folds"))
                go(at=put(at, s, "marked"), set_=mark, left=frozenset(range(S)) - {s})      # (the mark has got there before it looks)
            if at[s] == "marked":
                for o in left:
                    go(left=left - {o}, found=found if all(there[o]) else found | {o})
                if not left:
                    go(set_=sum(1 << o for o in found), at=put(at, s, "counts" if found else "folds"))
            if at[s] == "counts":
                add(s, -len(found), lib.come(count, -len(found)))
            if at[s] == "folds":
                assert "start" not in at
                if all(map(all, there)):
                    go(there=none, at=put(at, s, "done"), folds=folds + 1)
        if not new:
            assert (there, at, count, set_, folds) == (none, ("done",) * S, 0, 0, 1), state
            ends += 1
        for n in new:
            if n not in seen:
                seen.add(n)
                todo.append(n)
    assert ends >= 1
