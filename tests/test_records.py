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
extern "C" uint64_t come(uint64_t word, int s) { return after_coming(word, s); }
extern "C" uint64_t look(uint64_t word, uint64_t missed) { return after_looking(word, missed); }
extern "C" uint64_t mark() { return kLooking; }
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
    """All orders in which the slices of a row can send, their words and changes of the arrival word can take effect, and the last slice
    of few rows can give up, also before the others have started and however long a slice stays between two of its steps: one of
    them folds, after all have sent and with all words there, and words and arrival word are zero at the end, so that the next call
    finds nothing of this one.  (A record of two words here.)"""
    lib.mark.restype = lib.come.restype = lib.look.restype = C.c_uint64
    mark, come = lib.mark(), lambda v, s: lib.come(C.c_uint64(v), s)
    assert come(0, 5) == 0 and come(1 << 62, 62) == 0 and come(1 << 62, 61) == 1 << 62 and come(mark, 62) == mark | 1 << 62
    last, none, names = S - 1, ((False, False),) * S, ("there", "sent", "at", "seen_", "word", "left", "missed", "folds")
    # of each slice: its words that are there, its words that have got there, what it does next, the arrival word as it has seen it.
    # Then: the arrival word, and of the last slice: those it still has to look at, those it missed.  How often the row was folded.
    start = (none, none, ("start",) * S, (0,) * S, 0, frozenset(), frozenset(), 0)
    seen, todo, ends = {start}, [start], 0

    def put(t, s, v):
        return t[:s] + (v,) + t[s + 1:]
    while todo:
        state = todo.pop()
        there, sent, at, seen_, word, left, missed, folds = state
        new = []

        def go(**kw):
            new.append(tuple(kw.get(n, v) for n, v in zip(names, state)))
        for s in range(S):
            if at[s] == "start":
                go(at=put(at, s, "adds" if not few else "reads" if s == last else "waits"))
                continue
            for i in range(2):
                if not sent[s][i]:
                    go(there=put(there, s, put(there[s], i, True)), sent=put(sent, s, put(sent[s], i, True)))
            if at[s] == "adds":
                mine = lib.last(word, S)
                go(word=0 if mine else word + 1, at=put(at, s, "folds" if mine else "done"))
            if at[s] == "waits" and all(sent[s]):         # its record has got there: it looks at the word
                go(seen_=put(seen_, s, word), at=put(at, s, "done" if word == 0 else "comes"))
            if at[s] in ("comes", "leaves"):              # a compare-and-exchange, or a look at what stands there instead
                nxt = come(seen_[s], s) if at[s] == "comes" else lib.look(C.c_uint64(seen_[s]), C.c_uint64(sum(1 << o for o in missed)))
                if at[s] == "comes" and nxt == seen_[s]:
                    go(at=put(at, s, "done"))
                elif word == seen_[s]:
                    go(word=nxt, at=put(at, s, "done" if nxt else "folds"))
                else:
                    go(seen_=put(seen_, s, word))
            if at[s] == "reads":
                if all(map(all, there)):
                    go(at=put(at, s, "folds"))
                go(at=put(at, s, "looks"), word=mark, left=frozenset(range(S)) - {s})       # (the mark has got there before it looks)
            if at[s] == "looks":
                for o in left:
                    go(left=left - {o}, missed=missed if all(there[o]) else missed | {o})
                if not left:
                    go(seen_=put(seen_, s, mark), at=put(at, s, "leaves"))
            if at[s] == "folds":
                assert "start" not in at
                if all(map(all, there)):
                    go(there=none, at=put(at, s, "done"), folds=folds + 1)
        if not new:
            assert (there, at, word, folds) == (none, ("done",) * S, 0, 1), state
            ends += 1
        for n in new:
            if n not in seen:
                seen.add(n)
                todo.append(n)
    assert ends >= 1
