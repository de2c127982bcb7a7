// Device code of the Gumbel-max draws (Section 2.1.3: re-sampling from the adjusted distribution;
// generation loop of Algorithm 1: x_i ~ q_i), shared by the verification step's sampling kernel and
// by the drafting step: float keys that are upper bounds of the true keys, running winner and
// runner-up, and the float64 settlement of close calls.
#pragma once
#include "internal.h"
#include "noise_series.h"
#include "records.h"

namespace adasd {
namespace sampling {

constexpr float kErrRel = 1.52587890625e-05f;   // 2^-16: bound on the relative error of a float p or q
constexpr float kGuard = 1.220703125e-04f;      // 2^-13: bound on the log2-domain rounding of two keys

// Word (i & 3) of a Philox block by selects: indexing the array with a run-time value would make the
// compiler move it to LDS, and that lowering reads the dispatch packet for the workgroup size.
__device__ __forceinline__ uint32_t pick_word(const U4& r, int i) {
  const uint32_t lo = (i & 1) ? r.w[1] : r.w[0], hi = (i & 1) ? r.w[3] : r.w[2];
  return (i & 2) ? hi : lo;
}

__device__ __forceinline__ bool better(float ka, int ia, float kb, int ib) {
  return ka > kb || (ka == kb && (unsigned)ia < (unsigned)ib);
}

// Running winner (key, index) and the runner-up's KEY (its index is never needed).  One lane sees its
// elements in increasing index order, so a strict comparison keeps the lowest index on equal keys;
// across lanes `better` decides.  No branches.
__device__ __forceinline__ void top2_push(Top2& t, float k, int i) {
  const bool gt = k > t.k1;
  t.k2 = __builtin_amdgcn_fmed3f(k, t.k1, t.k2);     // (k1 >= k2: the middle one of the three is the new runner-up)
  t.i1 = gt ? i : t.i1;
  t.k1 = max_raw(t.k1, k);
}

__device__ __forceinline__ Top2 top2_merge(const Top2& a, const Top2& b) {
  const bool aw = better(a.k1, a.i1, b.k1, b.i1);
  Top2 r;
  r.k2 = fmaxf(fmaxf(a.k2, b.k2), aw ? b.k1 : a.k1);
  r.k1 = aw ? a.k1 : b.k1;
  r.i1 = aw ? a.i1 : b.i1;
  r.i2 = -1;
  return r;
}

// Wave-uniform result, given the best key of the wavefront: its lane by a ballot (the lowest index of all of them where
// several lanes hold that very key), then the best of what is left.
__device__ __forceinline__ Top2 top2_below(const Top2& v, float best) {
  Top2 r;
  r.i2 = -1;
  r.k1 = best;
  unsigned long long at = __ballot(v.k1 == r.k1);
  const int first = __ffsll((long long)at) - 1;
  r.i1 = __builtin_amdgcn_readlane(v.i1, first);
  if ((at & (at - 1)) == 0) {                                    // (uniform) one lane, the usual case
    r.k2 = wave_max_f((int)(threadIdx.x & 63) == first ? v.k2 : v.k1);
    return r;
  }
  r.k2 = r.k1;
  // (a wavefront without a logit, behind the end of a row or all masked, has -inf and no index in every lane: lane by lane it
  // took 1 us, and a row's slices wait for the slowest)
  if (__builtin_amdgcn_readfirstlane(__float_as_int(r.k1)) == (int)0xff800000) return r;
  while (at &= at - 1) {
    const int i = __builtin_amdgcn_readlane(v.i1, __ffsll((long long)at) - 1);
    r.i1 = (unsigned)i < (unsigned)r.i1 ? i : r.i1;
  }
  return r;
}
__device__ __forceinline__ Top2 top2_wave_reduce(const Top2& v) { return top2_below(v, wave_max_f(v.k1)); }

// log2 of -log2(u), u = (word + 0.5) / 2^32, i.e. log2 of E = -ln u up to a constant that every key shares: accurate
// to about 1e-6.  u is formed from the word and t = 1 - u from its complement, so that each is exact to a rounding
// where it is small (u as 1 - t would be 0 for the lowest 128 words).  The logarithm is u's, or where t is small
// the series of noise_series.h.
__device__ __forceinline__ float log2_exponential(uint32_t word) {
  const float u = fmaf((float)word, 0x1p-32f, 0x1p-33f), t = fmaf((float)(~word), 0x1p-32f, 0x1p-33f);
  const float series = log2_series(t), direct = lg2(u);
  return lg2(fabsf(t < kSerBelow ? series : direct));
}
// The same for the four words of a block, transcendentals in groups (device_common.h).
__device__ __forceinline__ void log2_exponential4(const U4& r, float (&lE)[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) lE[i] = fmaf((float)r.w[i], 0x1p-32f, 0x1p-33f);
  lg2_abs_group(lE);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float t = fmaf((float)(~r.w[i]), 0x1p-32f, 0x1p-33f), series = log2_series(t);
    lE[i] = t < kSerBelow ? series : lE[i];
  }
  lg2_abs_group(lE);
}

// Sampling modes of a sequence (SamplePlan::residual)
constexpr int kPlain = 0;      // the target row as it is (bonus row)
constexpr int kResidual = 1;   // max(0, p - q)
constexpr int kExclude = 2;    // the target row without one token (replacement after the loop's match test)

// Upper-bound key of one vocabulary element.
template <bool RESIDUAL>
__device__ __forceinline__ float key_ub(float zp, float zq, float cp, float cq, uint32_t word) {
  float lE = log2_exponential(word);
  if (!RESIDUAL) return fmaf(zp, kLog2e, -lE);         // log2 w = z log2 e + const
  float p = ex2(fmaf(zp, kLog2e, -cp)), q = ex2(fmaf(zq, kLog2e, -cq));
  float w = fmaxf(fmaf(kErrRel, p + q, p - q), 0.f);   // (p - q) + error bound; <= 0: certainly no mass
  return lg2(w) - lE;
}

// Hand-off of slice records inside one launch, by one wavefront of each workgroup: kXchgWords words per slice (records.h, which
// says who folds them).
// Where a row's slices leave their words: the first slots of its part of the hand-off region.
struct PlainWords {
  uint64_t* base;
  __device__ __forceinline__ uint64_t* at(int s) const { return base + s * kXchgWords; }
};
// The arrival words of the rows of a launch: a count each, or of few rows a set (64 bits), on a line of its own.
struct Arrivals {
  int32_t* base;
  int len, row, rows;
  __device__ __forceinline__ int32_t* count() const { return base + row * ticket_stride(rows, len); }                // (many rows)
  __device__ __forceinline__ uint64_t* set() const { return reinterpret_cast<uint64_t*>(base + row * 32); }          // (few rows)
};
static_assert(kFewRows * 32 <= kTicket1Len && kFewRows * 32 <= kTicket3Len, "a line of 128 bytes for each of few rows");
// (lane 0 adds 1; what the word held before, in every lane)
__device__ __forceinline__ int add_arrival(int32_t* word) {
  int before = 0;
  if ((threadIdx.x & 63) == 0) before = __hip_atomic_fetch_add(word, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return __builtin_amdgcn_readfirstlane(before);
}
// What this wavefront has stored has got there before anything is looked at that it loads from here on.
__device__ __forceinline__ void stores_before_loads() {
  publish_barrier();
  asm volatile("" ::: "memory");
}
template <class T> __device__ __forceinline__ void set_arrival(T* word, T v) {
  if ((threadIdx.x & 63) == 0) __hip_atomic_store(word, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t get_uniform(const uint64_t* word) {
  const uint64_t v = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return (uint64_t)(uint32_t)uniform((int)(v >> 32)) << 32 | (uint32_t)uniform((int)v);
}
// (lane 0 puts `next` in the place of `word`; where something else stood there, false, and word is what did)
__device__ __forceinline__ bool exchange_arrival(uint64_t* at, uint64_t& word, uint64_t next) {
  uint64_t seen = word;
  if ((threadIdx.x & 63) == 0)
    __hip_atomic_compare_exchange_strong(at, &seen, next, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  seen = (uint64_t)(uint32_t)uniform((int)(seen >> 32)) << 32 | (uint32_t)uniform((int)seen);
  const bool done = seen == word;
  word = seen;
  return done;
}
// The words of the lane's slice, and whether they are all there.
__device__ __forceinline__ bool look_at_words(const uint64_t* words, uint64_t (&w)[kXchgWords]) {
  bool there = true;
#pragma unroll
  for (int i = 0; i < kXchgWords; ++i) {
    w[i] = __hip_atomic_load(words + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    there = there && (w[i] & 1ull);
  }
  return there;
}
// Sends the record w of slice s of S > 1.  Returns whether this workgroup folds the row's records: then w has them, one slice per
// lane, all slices have sent, and words and arrival words are zero for the next launch.  slots.at(s): the words of slice s.
// ask(): what the one that folds asks for ahead of the wait.  arrived: false where the records have been sent and still do not
// come: calls that share a workspace have not been ordered, and one has cleared the other's words.  The caller then goes by the
// logits themselves.
// (What a slice of few rows does behind its record stands beside the last slice's wait and shows in no call's time.  With one count
// for them all, which every slice adds to, it did: one after the other, the returned additions were what the kernel ended with,
// 1 x 8 x 128256 bf16 14.9 -> 15.3 us a call; and so did records sent by an exchange, 32 x 128256 float 6.2 -> 7.3.  Giving a row up stands behind
// the wait and not in its loop, where it lay in the way: 1 x 8 x 128256 15.0 -> 14.9.)
template <class Slots, class Ask>
__device__ __forceinline__ bool hand_off(const Slots& slots, int s, int S, const Arrivals& a, WordWait wait, const Ask& ask,
                                         uint64_t (&w)[kXchgWords], bool& arrived) {
  const int lane = threadIdx.x & 63;
  const uint64_t w0 = w[0], w1 = w[1], w2 = w[2], word = lane == 0 ? w0 : lane == 1 ? w1 : w2;
  static_assert(kXchgWords == 3, "a lane per word");
  if (lane < kXchgWords) __hip_atomic_store(slots.at(s) + lane, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const bool may_give_up = few_rows(a.rows) && s == S - 1;
  if (!may_give_up) {
    if (!few_rows(a.rows)) {
      if (!last_to_add(add_arrival(a.count()), S)) return false;
      set_arrival(a.count(), 0);
    } else {
      stores_before_loads();
      uint64_t set = get_uniform(a.set()), next;
      if (__builtin_expect(set == 0, 1)) return false;
      do {
        next = after_coming(set, s);
        if (next == set) return false;
      } while (!exchange_arrival(a.set(), set, next));
      if (next != 0) return false;
    }
  }
  ask();
  const bool mine = lane < S;
  uint64_t* words = slots.at(min(lane, S - 1));
  auto wait_for_words = [&](int polls) {
    bool there;
    do there = __all(look_at_words(words, w) || !mine) != 0;
    while (!there && polls-- > 0);
    return there;
  };
  arrived = wait_for_words(may_give_up && wait == kGivesUp ? 0 : kWaitPolls);
  if (__builtin_expect(!arrived && may_give_up, 0)) {
    set_arrival(a.set(), kLooking);
    stores_before_loads();
    const uint64_t missed = __ballot(mine && lane != s && !look_at_words(words, w));
    uint64_t set = kLooking, next;
    do next = after_looking(set, missed);
    while (!exchange_arrival(a.set(), set, next));
    if (next != 0) return false;
    arrived = wait_for_words(kWaitPolls);
  }
  if (mine) {
#pragma unroll
    for (int i = 0; i < kXchgWords; ++i) __hip_atomic_store(words + i, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (wait == kNotThere) arrived = false;
  return true;
}

// ---- logits that cannot win any more: the two logarithms of a logit's noise are only formed where its bound
// (noise_series.h) comes up to `floor`, a lower bound (less kReach) of the true key of an element that was looked at.  Of the
// n-th group of exchangeable logits that is one in n.  An element left out lies under the floor by more than the guard: it is
// not the winner, and neither the winner nor whether it needs settling in float64 (a runner-up within the margin,
// another element at or above the winner's lower bound) depends on it.
// The factor that takes 2^(key without noise, less `of`) to the scale of the noise words.
__device__ __forceinline__ float reach(float of, float floor) { return ex2(reach_exponent(of - floor)); }
// Whether any lane's group of four may hold an element that reaches the floor.  (NaN: yes.)
__device__ __forceinline__ bool may_win(const float (&e)[4], float f, const U4& block) {
  float v[4], top;
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = noise_reach(e[i], f, block.w[i]);
  asm("v_maximum3_f32 %0, %1, %2, %3" : "=v"(top) : "v"(v[0]), "v"(v[1]), "v"(v[2]));
  asm("v_maximum3_f32 %0, %0, %1, %1" : "+v"(top) : "v"(v[3]));
  return __any(!(top <= kNoiseTop)) != 0;
}

// The floors of a workgroup's wavefronts, in shared memory: each turn starts from the highest.  (Which of them a wavefront
// comes to see decides what it leaves out, and nothing else.)
struct Floors {
  float f[kWaves];
};
__device__ __forceinline__ void floors_init(Floors& sh) {
  if (threadIdx.x < kWaves) sh.f[threadIdx.x] = kNoFloor;
  __syncthreads();
}
__device__ __forceinline__ float highest_floor(const Floors& sh, float mine) {
#pragma unroll
  for (int w = 0; w < kWaves; ++w)
    mine = fmaxf(mine, __hip_atomic_load(&sh.f[w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
  return mine;
}
__device__ __forceinline__ float raise_floor(Floors& sh, float mine, float lane_floor) {
  mine = fmaxf(mine, wave_max_f(floor_of(lane_floor)));
  __hip_atomic_store(&sh.f[__builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6)], mine, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_WORKGROUP);        // (every lane the same)
  return mine;
}

// Four logits (group g of a vector, the first of index `first`) with their block of noise.  PRUNE: those that cannot win
// are left out (floor, uniform: see above).
template <int DT, int MODE, bool PRUNE>
__device__ __forceinline__ void scan_group(const uint4& xp, const uint4& xq, int g, int first, const U4& block, float neg_cp,
                                           float neg_cq, int excluded, Top2& best, Floors& sh, float& floor, bool& poison) {
  float zp[4], e[4], lE[4], lane_floor = -INFINITY;
  unpack4<DT>(xp, g, zp);
  if (MODE == kResidual) {
    float zq[4], p[4], q[4];
    unpack4<DT>(xq, g, zq);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      zp[i] = fma_log2e(zp[i], neg_cp);
      zq[i] = fma_log2e(zq[i], neg_cq);
    }
    ex2_group(zp, p);
    ex2_group(zq, q);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      zq[i] = kErrRel * (p[i] + q[i]);                       // (the error of the difference)
      e[i] = max_raw(zq[i] + (p[i] - q[i]), 0.f);
    }
    if (PRUNE) {
      if (!may_win(e, reach(0.f, floor), block)) return;
#pragma unroll
      for (int i = 0; i < 4; ++i) {                          // (how far the true key may lie below: see the margin in k_sample)
        const float w = e[i] - zq[i];
        zq[i] = w > 2.f * zq[i] ? 3.f * kLog2e * zq[i] * __builtin_amdgcn_rcpf(w) : INFINITY;
      }
    }
    lg2_abs_group(e);
    log2_exponential4(block, lE);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float k = e[i] - lE[i];
      if (PRUNE) lane_floor = max_raw(lane_floor, k - zq[i]);
      top2_push(best, k, first + i);
    }
  } else {
    if (PRUNE) {
      float t[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) t[i] = fma_log2e(zp[i], -floor);
      ex2_group(t, e);
      if (!may_win(e, 1.f, block)) return;
    }
    log2_exponential4(block, lE);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (MODE == kPlain) poison |= !(zp[i] < INFINITY);       // NaN or +inf in the bonus row
      float k = fma_log2e(zp[i], -lE[i]);
      if (MODE == kExclude) k = first + i == excluded ? -INFINITY : k;
      top2_push(best, k, first + i);
    }
    lane_floor = best.k1;
  }
  if (PRUNE) floor = raise_floor(sh, floor, lane_floor);
}

// ---- the scan of one slice ----------------------------------------------------------------------
// Vectors v0 .. v1 of the row(s), one per thread and turn, the next one always on its way.  col0: vocabulary index of
// the row's first element (0 unless the row is a column slice; a multiple of eight); indices, the excluded token
// and the noise counters are in vocabulary indices.
// Bound by the vector ALU as the drafting kernel is (draft.hip); the whole round against the scan in batches of two
// vectors: 128 x 16 x 152064 385 -> 376 us, ragged 64 x 16 x 128256 127 -> 116 us, 32 x 8 x 128256 64.8 -> 62.2 us (the
// same statistics kernel in both).  With PRUNE, the token kernel alone: 128 x 16 x 152064 28.2 -> 24.4 us, ragged
// 64 x 16 x 128256 15.0 -> 14.3 us.
// kExclude gives a key to every finite logit but the excluded one, also to those whose probability is 0
// in float64 (which the float64 path skips).  Such an element cannot win: this mode only runs after the
// match test rejected the excluded token x, i.e. ln u1 >= ln p(x) with u1 < 1 - 2^-25, so the rest of the
// row holds a mass of at least 3e-8 and some element at least 3e-8 / V of it; its key is above -50 nats
// whatever its noise, the key of an element with p < 5e-324 below -720.
template <int DT, int MODE, bool PRUNE>
__device__ __forceinline__ void scan_slice(const char* prow, const char* qrow, int V, int v0, int v1, float cp, float cq,
                                           int excluded, int col0, const PhiloxRow& noise, Top2& best, Floors& sh, bool& poison) {
  constexpr bool RESIDUAL = MODE == kResidual;
  constexpr int EPV = Elem<DT>::per_vec;
  const int tid = threadIdx.x, whole = V / EPV;
  auto load = [&](const char* row, int idx) {
    uint4 x = neutral_vec<DT>();
    if (idx < v1) {
      if (idx < whole) x = load_vec_any(row, idx);
      else x = load_last_vec<DT>(row, V);
    }
    return x;
  };
  float neg_cp = -cp, neg_cq = -cq, floor = kNoFloor;
  asm volatile("" : "+v"(neg_cp), "+v"(neg_cq));
  uint4 next_p = load(prow, v0 + tid), next_q = next_p;
  if (RESIDUAL) next_q = load(qrow, v0 + tid);
  for (int base = v0; base < v1; base += kBlock) {
    const uint4 xp = next_p, xq = next_q;
    const int idx = base + tid;
    if (base + kBlock < v1) {
      next_p = load(prow, idx + kBlock);
      if (RESIDUAL) next_q = load(qrow, idx + kBlock);
    }
    if (base + (tid & ~63) >= v1) continue;     // (a whole wavefront past the end)
    if (PRUNE) floor = highest_floor(sh, floor);
#pragma unroll
    for (int g = 0; g < EPV / 4; ++g) {
      const int first = col0 + idx * EPV + 4 * g;
      scan_group<DT, MODE, PRUNE>(xp, xq, g, first, philox_block(noise, (uint32_t)first >> 2), neg_cp, neg_cq, excluded, best, sh, floor, poison);
    }
  }
}

// The same where a long row has no more than its slices on the chip, one wavefront to a SIMD: sixteen logits per thread
// and turn, whose noise is formed ahead of the rest, so that the chains of four Philox blocks fill each other's gaps.
template <int DT, int MODE, bool PRUNE>
__device__ __forceinline__ void scan_long_slice(const char* prow, const char* qrow, int V, int v0, int v1, float cp, float cq,
                                                int excluded, const PhiloxRow& noise, Top2& best, Floors& sh, bool& poison) {
  constexpr bool RESIDUAL = MODE == kResidual;
  constexpr int EPV = Elem<DT>::per_vec, G = EPV / 4, NV = 4 / G;
  const int tid = threadIdx.x, whole = V / EPV;
  // (requested without a branch: between loads that may or may not be made the compiler waits for the one before)
  uint4 next_p[NV], next_q[NV];
  auto request = [&](int base) {
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const int idx = min(base + tid + j * kBlock, whole - 1);
      next_p[j] = load_vec_any(prow, idx);
      if (RESIDUAL) next_q[j] = load_vec_any(qrow, idx);
    }
  };
  auto settle = [&](const char* row, int idx, const uint4& x) {     // what stands there: past the slice's end -inf in every logit
    const uint4 none = neutral_vec<DT>();
    const bool in = idx < v1;
    uint4 y = make_uint4(in ? x.x : none.x, in ? x.y : none.y, in ? x.z : none.z, in ? x.w : none.w);
    if (in && idx == whole) y = load_last_vec<DT>(row, V);
    return y;
  };
  float floor = kNoFloor;
  request(v0);
  for (int base = v0; base < v1; base += NV * kBlock) {
    uint4 xp[NV], xq[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      xp[j] = xq[j] = settle(prow, base + tid + j * kBlock, next_p[j]);
      if (RESIDUAL) xq[j] = settle(qrow, base + tid + j * kBlock, next_q[j]);
    }
    if (base + NV * kBlock < v1) request(base + NV * kBlock);
    if (base + (tid & ~63) >= v1) continue;     // (a whole wavefront past the end)
    if (PRUNE) floor = highest_floor(sh, floor);
    U4 block[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) block[j] = philox_block(noise, (uint32_t)((base + tid + j / G * kBlock) * EPV + j % G * 4) >> 2);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      scan_group<DT, MODE, PRUNE>(xp[j / G], xq[j / G], j % G, (base + tid + j / G * kBlock) * EPV + j % G * 4, block[j], -cp, -cq, excluded,
                           best, sh, floor, poison);
  }
}

// ---- float64 re-evaluation of one sequence by one workgroup ------------------------------------
__device__ inline double block_max_d(double v, double* sh) {
  v = wave_max(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = sh[0];
#pragma unroll
  for (int w = 1; w < kWaves; ++w) t = fmax(t, sh[w]);
  return t;
}
__device__ inline double block_sum_d(double v, double* sh) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) t += sh[w];
  return t;
}

template <int DT>
__device__ double row_lse_exact(const char* row, int V, double* sh) {
  double m = -INFINITY;
  for (int v = threadIdx.x; v < V; v += kBlock) m = fmax(m, (double)load_elem<DT>(row, v));
  m = block_max_d(m, sh);
  if (!(m > -INFINITY)) return NAN;
  double s = 0.0;
  for (int v = threadIdx.x; v < V; v += kBlock) s += exp((double)load_elem<DT>(row, v) - m);
  s = block_sum_d(s, sh);
  return m + log(s);
}

// Returns the token (all threads), -1 if the row has no finite logit.
template <int DT>
__device__ __forceinline__ int sample_exact(const char* prow, const char* qrow, bool residual, int excluded, int V, uint32_t c1,
                            uint32_t c2, uint32_t c3, uint32_t k0, uint32_t k1, double* sh,
                            uint32_t* status_bits) {
  const double lse_p = row_lse_exact<DT>(prow, V, sh);
  if (isnan(lse_p)) {
    *status_bits |= ADASD_ST_NONFINITE;
    return -1;
  }
  double lse_q = 0.0;
  if (residual) {
    lse_q = row_lse_exact<DT>(qrow, V, sh);
    double mass = 0.0;
    for (int v = threadIdx.x; v < V; v += kBlock) {
      double w = exp((double)load_elem<DT>(prow, v) - lse_p) - exp((double)load_elem<DT>(qrow, v) - lse_q);
      if (w > 0.0) mass += w;
    }
    mass = block_sum_d(mass, sh);
    if (!(mass > 0.0)) {           // no residual mass: the token comes from the target distribution
      residual = false;
      *status_bits |= ADASD_ST_ZERO_MASS;
    }
  }
  if (excluded >= 0) {
    double mass = 0.0;
    for (int v = threadIdx.x; v < V; v += kBlock)
      if (v != excluded) mass += exp((double)load_elem<DT>(prow, v) - lse_p);
    mass = block_sum_d(mass, sh);
    if (!(mass > 0.0)) {           // everything sits on the excluded token: the target row as it is
      excluded = -1;
      *status_bits |= ADASD_ST_ZERO_MASS;
    }
  }
  double best = -INFINITY;
  int tok = 0x7fffffff;
  for (int v = threadIdx.x; v < V; v += kBlock) {
    double w = exp((double)load_elem<DT>(prow, v) - lse_p);
    if (residual) w -= exp((double)load_elem<DT>(qrow, v) - lse_q);
    if (v == excluded || !(w > 0.0)) continue;
    const U4 r = philox4x32_10((uint32_t)v >> 2, c1, c2, c3, k0, k1);
    const double u = ((double)pick_word(r, v) + 0.5) * (1.0 / 4294967296.0);
    const double key = log(w) - log(-log(u));
    if (key > best) {               // v increases per thread: the first index keeps a tie
      best = key;
      tok = v;
    }
  }
  // block argmax with lowest index on equal keys
  const double bmax = block_max_d(best, sh);
  int cand = (best == bmax && tok != 0x7fffffff) ? tok : 0x7fffffff;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) cand = min(cand, __shfl_xor(cand, off));
  __shared__ int sh_tok[kWaves];
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh_tok[threadIdx.x >> 6] = cand;
  __syncthreads();
  int t = sh_tok[0];
#pragma unroll
  for (int w = 1; w < kWaves; ++w) t = min(t, sh_tok[w]);
  return t == 0x7fffffff ? -1 : t;
}

// Vectors per slice of a row of nv vectors cut into S slices: equal shares, in whole 128-byte lines where the last
// slice then still has work.
__host__ __device__ inline int slice_chunk(int nv, int S) {
  const int even = (nv + S - 1) / S, lines = (even + 7) / 8 * 8;
  return (int64_t)lines * (S - 1) < nv ? lines : even;
}

constexpr int kMaxCand = 64;      // elements that may still win
constexpr int kMaxRescan = 8;     // slices that hold more than one of them

struct RefineShared {
  int n_cand, n_rescan;
  int cand[kMaxCand];
  int rescan[kMaxRescan];
  double key[kMaxCand], err[kMaxCand];
  int result;                     // token, or -1: too close, the whole row is needed
};

// Normaliser of a row to float64 accuracy in the arguments and one float ulp per term: sum of
// 2^(z log2 e - c) around a first value c of the normaliser, each term the hardware exponential of the
// float part of the argument times the first-order factor of the remainder.  Returns ln sum exp z.
// (the sum itself, all threads get it: column shards add theirs up before the logarithm)
template <int DT>
__device__ double row_pow2_sum_refined(const char* row, int V, double c_lse2, double* sh) {
  constexpr int EPV = Elem<DT>::per_vec;
  auto term = [&](float z) {
    const double x = (double)z * 1.44269504088896340736 - c_lse2;
    const float xf = (float)x;
    return xf > -140.f ? (double)ex2(xf) * (1.0 + (x - (double)xf) * 0.69314718055994530942) : 0.0;
  };
  const int tid = threadIdx.x;
  double acc = 0.0;
  // one workgroup walks the whole row: several vectors per thread in flight, or the latency of each
  // load is paid in full
  const int nv = (reinterpret_cast<uintptr_t>(row) & 15u) == 0 ? V / EPV : 0;
  const uint4* vp = reinterpret_cast<const uint4*>(row);
  constexpr int NB = 2;   // more would raise the register count of every kernel this is inlined into
  for (int base = 0; base < nv; base += NB * kBlock) {
    uint4 x[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) x[j] = vp[min(base + tid + j * kBlock, nv - 1)];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      float z[EPV];
      unpack<DT>(x[j], z);
      double part = 0.0;
#pragma unroll
      for (int e = 0; e < EPV; ++e) part += term(z[e]);
      if (base + tid + j * kBlock < nv) acc += part;
    }
  }
  for (int v = nv * EPV + tid; v < V; v += kBlock) acc += term(load_elem<DT>(row, v));
  return block_sum_d(acc, sh);
}
template <int DT>
__device__ double row_lse_refined(const char* row, int V, double c_lse2, double* sh) {
  const double acc = row_pow2_sum_refined<DT>(row, V, c_lse2, sh);
  return (c_lse2 + log(acc) * 1.44269504088896340736) * 0.69314718055994530942;
}

// Collects into R.cand the elements (vocabulary indices) whose upper-bound key is at least tau, from the
// per-slice records of the scan (a slice whose runner-up also reaches tau is scanned again).  All threads
// of the workgroup call it; false: more candidates or slices than the lists hold.  col0: vocabulary index
// of the row's first element (the rows are column slices of V elements when it is not 0).
template <int DT>
__device__ bool refine_gather(const char* prow, const char* qrow, bool residual, int excluded, int V, int col0, int b,
                              int S, float tau, float cp, float cq, uint32_t c1, uint32_t c2, uint32_t c3,
                              uint32_t k0, uint32_t k1, const Workspace& ws, RefineShared& R) {
  const int tid = threadIdx.x;
  if (tid == 0) R.n_cand = R.n_rescan = 0;
  __syncthreads();
  // per-slice records: the slice's best element if it reaches tau; the slice itself if its runner-up does
  for (int j = tid; j < S; j += kBlock) {
    const Top2* src = &ws.part3[(size_t)b * kMaxSampleSplit + j];
    const float s_k1 = ld_agent(&src->k1), s_k2 = ld_agent(&src->k2);
    const int s_i1 = ld_agent(&src->i1);
    if (s_k2 >= tau) {
      const int at = atomicAdd(&R.n_rescan, 1);
      if (at < kMaxRescan) R.rescan[at] = j;
    } else if (s_k1 >= tau && s_i1 >= 0) {
      const int at = atomicAdd(&R.n_cand, 1);
      if (at < kMaxCand) R.cand[at] = s_i1;
    }
  }
  __syncthreads();
  const int n_rescan = R.n_rescan;
  if (n_rescan > kMaxRescan) return false;
  const int width = slice_chunk(vectors_of<DT>(V), S) * Elem<DT>::per_vec;    // logits per slice
  for (int n = 0; n < n_rescan; ++n) {
    const int lo = min(R.rescan[n] * width, V), hi = min(lo + width, V);
    for (int v = lo + tid; v < hi; v += kBlock) {
      const int gv = col0 + v;
      const U4 r = philox4x32_10((uint32_t)gv >> 2, c1, c2, c3, k0, k1);
      const float zp = load_elem<DT>(prow, v);
      const float k = residual ? key_ub<true>(zp, load_elem<DT>(qrow, v), cp, cq, pick_word(r, gv))
                               : key_ub<false>(zp, 0.f, cp, cq, pick_word(r, gv));
      if (k >= tau && gv != excluded) {
        const int at = atomicAdd(&R.n_cand, 1);
        if (at < kMaxCand) R.cand[at] = gv;
      }
    }
  }
  __syncthreads();
  return R.n_cand <= kMaxCand;
}

// Settles a sequence among the elements whose upper-bound key is at least tau.  All threads of the
// workgroup call it; returns the token, or -1 if the decision needs the whole row in float64.
template <int DT>
__device__ __forceinline__ int sample_refine(const char* prow, const char* qrow, int mode, int excluded, int V, int b, int S,
                             float tau, float cp, float cq, double lse2_p, double lse2_q, uint32_t c1,
                             uint32_t c2, uint32_t c3, uint32_t k0, uint32_t k1, const Workspace& ws,
                             double* sh_red, RefineShared& R) {
  const int tid = threadIdx.x;
  const bool residual = mode == kResidual;
  if (!refine_gather<DT>(prow, qrow, residual, excluded, V, 0, b, S, tau, cp, cq, c1, c2, c3, k0, k1, ws, R)) return -1;
  const int n_cand = R.n_cand;
  if (n_cand == 0) return -1;
  // float64 keys of the candidates.  Without a draft row the normaliser is a common shift and drops
  // out; with it both normalisers are refined first (workgroup-wide), and each key carries the bound
  // 2^-21 (p + q) / w of what their remaining error can do to ln w.
  double lse_p = 0.0, lse_q = 0.0;
  if (residual) {
    lse_p = row_lse_refined<DT>(prow, V, lse2_p, sh_red);
    lse_q = row_lse_refined<DT>(qrow, V, lse2_q, sh_red);
  }
  if (tid < n_cand) {
    const int v = R.cand[tid];
    const U4 r = philox4x32_10((uint32_t)v >> 2, c1, c2, c3, k0, k1);
    const double u = ((double)pick_word(r, v) + 0.5) * (1.0 / 4294967296.0);
    const double g = log(-log(u));
    double key, err = 0.0;
    if (residual) {
      const double p = exp((double)load_elem<DT>(prow, v) - lse_p), q = exp((double)load_elem<DT>(qrow, v) - lse_q);
      const double w = p - q;
      err = w > 0.0 ? 0x1p-21 * (p + q) / w : INFINITY;
      key = w > 0.0 ? log(w) - g : -INFINITY;
    } else {
      key = (double)load_elem<DT>(prow, v) - g;
    }
    R.key[tid] = key;
    R.err[tid] = err;
  }
  __syncthreads();
  if (tid == 0) {
    int best = 0;
    for (int c = 1; c < n_cand; ++c)
      if (R.key[c] > R.key[best] || (R.key[c] == R.key[best] && R.cand[c] < R.cand[best])) best = c;
    int result = R.cand[best];
    if (residual) {
      // final only if no other candidate can overtake within the error bounds; a candidate whose mass
      // is not certain at this accuracy sends the sequence to the whole-row path
      if (!(R.err[best] < 0.25)) result = -1;
      for (int c = 0; c < n_cand && result >= 0; ++c) {
        if (c == best) continue;
        if (!(R.err[c] < 0.25)) result = -1;
        else if (!(R.key[best] - R.err[best] > R.key[c] + R.err[c])) result = -1;
      }
    }
    R.result = result;
  }
  __syncthreads();
  return R.result;
}

}  // namespace sampling
}  // namespace adasd
