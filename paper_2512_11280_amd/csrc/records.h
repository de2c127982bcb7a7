// Slice records as they travel between the workgroups of one launch: 64-bit words of two 32-bit halves, each of which
// says itself that it is there (bit 0 of its low half is set in every record; cleared words are 0).  A record
// arrives as it was sent, to the last bit: where a float gives its lowest bit to the flag, that bit travels elsewhere
// in the record.  Nothing but bit arithmetic, so that the CPU tests compile this file as it is.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#define ADASD_ANYWHERE __host__ __device__ __forceinline__
#else
#define ADASD_ANYWHERE inline
#endif

namespace adasd {

ADASD_ANYWHERE uint32_t bits_of(float v) {
  uint32_t b;
  __builtin_memcpy(&b, &v, 4);
  return b;
}
ADASD_ANYWHERE float float_of(uint32_t b) {
  float v;
  __builtin_memcpy(&v, &b, 4);
  return v;
}

ADASD_ANYWHERE uint64_t record_word(uint32_t lo, float hi) { return ((uint64_t)bits_of(hi) << 32) | lo; }
ADASD_ANYWHERE float word_hi(uint64_t w) { return float_of((uint32_t)(w >> 32)); }
ADASD_ANYWHERE float word_lo(uint64_t w) { return float_of((uint32_t)w); }
ADASD_ANYWHERE uint32_t word_index(int i) { return (uint32_t)(i + 2) * 2u + 1u; }
ADASD_ANYWHERE int index_of_word(uint64_t w) { return (int)((uint32_t)w >> 1) - 2; }

// A slice of the token kernel: best key and its index, runner-up key, whether a broken logit was met, the logits of the
// best (the error of its key is formed from them, and has to be the same however the row is cut).
struct DrawRecord {
  float k1, k2, zp, zq;
  int i1;
  bool poison;
};
ADASD_ANYWHERE void pack_draw(const DrawRecord& r, uint64_t (&w)[3]) {
  w[0] = record_word(word_index(r.i1), r.k1);
  w[1] = record_word(1u | (r.poison ? 2u : 0u) | ((bits_of(r.zp) & 1u) << 2), r.k2);
  w[2] = record_word(bits_of(r.zp) | 1u, r.zq);
}
ADASD_ANYWHERE DrawRecord unpack_draw(const uint64_t (&w)[3]) {
  DrawRecord r;
  r.k1 = word_hi(w[0]);
  r.i1 = index_of_word(w[0]);
  r.k2 = word_hi(w[1]);
  r.poison = ((uint32_t)w[1] & 2u) != 0;
  r.zp = float_of(((uint32_t)w[2] & ~1u) | (((uint32_t)w[1] >> 2) & 1u));
  r.zq = word_hi(w[2]);
  return r;
}

// A weighted sum u whose word also holds the flag: its lowest bit travels as the sign of the sum s, which has none.
ADASD_ANYWHERE float sum_with_bit(float s, float u) { return float_of((bits_of(s) & 0x7fffffffu) | (bits_of(u) << 31)); }
ADASD_ANYWHERE float sum_alone(float s) { return float_of(bits_of(s) & 0x7fffffffu); }
ADASD_ANYWHERE float flagged(float u) { return float_of(bits_of(u) | 1u); }
ADASD_ANYWHERE float with_bit_of(float u, float s) { return float_of((bits_of(u) & ~1u) | (bits_of(s) >> 31)); }

// A slice of the drafting kernel: reference (whose lowest bit is set, the sums being formed about such a one), sum of
// exponentials (>= 0, or NaN), weighted sum; best key and its index, runner-up key.
struct DraftRecord {
  float m, s, u, k1, k2;
  int i1;
};
ADASD_ANYWHERE void pack_draft(const DraftRecord& r, uint64_t (&w)[3]) {
  w[0] = record_word(bits_of(r.m), sum_with_bit(r.s, r.u));
  w[1] = record_word(bits_of(flagged(r.u)), r.k1);
  w[2] = record_word(word_index(r.i1), r.k2);
}
ADASD_ANYWHERE DraftRecord unpack_draft(const uint64_t (&w)[3]) {
  DraftRecord r;
  r.m = word_lo(w[0]);
  r.s = sum_alone(word_hi(w[0]));
  r.u = with_bit_of(word_lo(w[1]), word_hi(w[0]));
  r.k1 = word_hi(w[1]);
  r.i1 = index_of_word(w[2]);
  r.k2 = word_hi(w[2]);
  return r;
}

// A slice of a row pair in the statistics kernel: target row (p) and draft row (q), references with their lowest bit set.
struct PairRecord {
  float mp, sp, up, mq, sq, uq;
};
ADASD_ANYWHERE void pack_pair(const PairRecord& r, uint64_t (&w)[3]) {
  w[0] = record_word(bits_of(r.mp), sum_with_bit(r.sp, r.up));
  w[1] = record_word(bits_of(r.mq), r.sq);
  w[2] = record_word(bits_of(flagged(r.up)), r.uq);
}
ADASD_ANYWHERE PairRecord unpack_pair(const uint64_t (&w)[3]) {
  return PairRecord{word_lo(w[0]), sum_alone(word_hi(w[0])), with_bit_of(word_lo(w[2]), word_hi(w[0])),
                    word_lo(w[1]), word_hi(w[1]), word_hi(w[2])};
}

// Who folds the records of a row of S > 1 slices, by the row's arrival word (zero between launches).
//  * Many rows: a count.  Every slice sends its record and adds 1.  The last one to add folds: all records have been sent by
//    then, and it reads until they are there.
//  * Few rows: the last slice reads at once, which saves it a round trip.  Should it read for too long (those it waits for may
//    not have been started, if work of other streams holds the chip) it gives up: it puts kLooking in the word and, when that
//    has got there, looks once more.  A slice looks at the word when its record has got there; so one that still finds zero
//    has its record found.  One that finds kLooking adds itself to the word, and need not be waited for any more.  The last slice then
//    puts in the place of kLooking the slices whose records it has missed and that have not come meanwhile; they take themselves out
//    again as they come.  Whoever leaves zero is the last and folds.  Each change is one compare-and-exchange, begun again where
//    the word has changed meanwhile: nobody waits for anybody, and a word changes no more often than there are slices.
// Either way all slices have sent before anybody folds, clears words or changes a state, and no word is left behind.
ADASD_ANYWHERE bool last_to_add(int before, int S) { return before == S - 1; }             // many rows
constexpr uint64_t kLooking = 1ull << 63;                                                   // (the last slice of 64 is in no set)
ADASD_ANYWHERE bool being_looked(uint64_t word) { return (word & kLooking) != 0; }
// What a slice makes of the word, its record being there (the word itself: nothing is to be done), and whether it then folds.
ADASD_ANYWHERE uint64_t after_coming(uint64_t word, int s) {
  const uint64_t self = 1ull << s;
  return word == 0 ? 0 : being_looked(word) ? word | self : word & ~self;
}
// What the last slice makes of it, having missed the records of these slices.  (It folds where that leaves zero.)
ADASD_ANYWHERE uint64_t after_looking(uint64_t word, uint64_t missed) { return missed & ~word; }

}  // namespace adasd
