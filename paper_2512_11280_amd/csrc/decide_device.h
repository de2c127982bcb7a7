// Device code of the acceptance decisions of one sequence (Section 2.1.3, Section 4.4 and the
// verification loop of Algorithm 1 of the paper) and of the update step.
#pragma once
#include "history_device.h"

namespace adasd {

// The lists hold distances strictly inside (d_eps, 1 - d_eps) (Section 4.4 leaves out the values "exactly 0
// or 1").  1 - d is exact in float from d = 1/2 on, so this is the comparison of the real numbers; 1 - d_eps
// rounded to float would shut out the float just below it.  NaN fails both.
__device__ __forceinline__ bool inside_open_interval(float d, float d_eps) { return d > d_eps && 1.0f - d > d_eps; }

constexpr int kHalfU = 4;      // samples per lane in flight where 32 lanes walk a list

// Sums of x - c and of its square over a list, by 32 lanes.
__device__ __forceinline__ void half_moments(const float* L, int n, double c, double& s1, double& s2) {
  const int l32 = threadIdx.x & 31;
  s1 = s2 = 0.0;
#pragma unroll 1
  for (int base = 0; base < n; base += 32 * kHalfU) {
    float x[kHalfU];
#pragma unroll
    for (int u = 0; u < kHalfU; ++u) x[u] = L[min(base + l32 + 32 * u, n - 1)];
#pragma unroll
    for (int u = 0; u < kHalfU; ++u) {
      const double e = base + l32 + 32 * u < n ? (double)x[u] - c : 0.0;
      s1 += e;
      s2 += e * e;
    }
  }
  s1 = half_sum_d(s1);
  s2 = half_sum_d(s2);
}

// Sums of x - c and of its square over the nx <= 64 samples of X, by 32 lanes, onto s1 and s2.
__device__ __forceinline__ void add_moments(const float* X, int nx, double c, double& s1, double& s2) {
  const int l32 = threadIdx.x & 31;
  const double e0 = l32 < nx ? (double)X[l32] - c : 0.0, e1 = l32 + 32 < nx ? (double)X[l32 + 32] - c : 0.0;
  s1 += half_sum_d(e0 + e1);
  s2 += half_sum_d(e0 * e0 + e1 * e1);
}

// A batch of a list's samples joins a thread's running sum of kernels: acc * 2^m, where m is the largest exponent so far.
// An exponent is rounded before the reference is taken from it, as the reference was, so that the nearest sample counts as 1
// exactly: a list whose samples agree to an ulp has exponents of -1e20, where one rounding is 1e4.  (Product and reference in
// one fma, the nearest sample found by its distance: an instruction less per sample and the same time, 128 x 16 positions with
// lists of 4000 53.0 us a round either way, 32 x 8 30.6, 128 x 16 with lists of 448 41.1.)  Samples that do not count are infinite.
template <int N, class Sum>
__device__ __forceinline__ void join_kernels(double d, const float (&x)[N], double scale, double& m, Sum& acc) {
  double t[N], hi = m;
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const double e = d - (double)x[u];
    t[u] = -(e * e) * scale;
    hi = fmax(hi, t[u]);
  }
  const double ref = hi > -INFINITY ? hi : 0.0;            // (nothing to add yet: every factor is 2^-inf = 0)
  float add = 0.f;
#pragma unroll
  for (int u = 0; u < N; ++u) add += ex2((float)(t[u] - ref));    // terms below 2^-126 vanish
  acc = acc * (Sum)ex2((float)(m - ref)) + (Sum)add;
  m = hi;
}

// log2 [ p(d | list) P(list) ] by 32 lanes.  EXTRA: the list goes on in X (nx <= 64 samples); else head holds the lane's first ones.
template <bool EXTRA>
__device__ __forceinline__ double half_log_joint(double d, const float* L, const float (&head)[kHalfU], int n, const float* X, int nx,
                                                 const Kde& k) {
  const int l32 = threadIdx.x & 31;
  double m = -INFINITY;
  float acc = 0.f;
  if (!EXTRA) {
    float x[kHalfU];
#pragma unroll
    for (int u = 0; u < kHalfU; ++u) x[u] = l32 + 32 * u < n ? head[u] : INFINITY;
    join_kernels(d, x, k.scale, m, acc);
  }
#pragma unroll 1
  for (int base = l32 + (EXTRA ? 0 : 32 * kHalfU); base - l32 < n; base += 32 * kHalfU) {
    float x[kHalfU];
#pragma unroll
    for (int u = 0; u < kHalfU; ++u) x[u] = L[min(base + 32 * u, n - 1)];
#pragma unroll
    for (int u = 0; u < kHalfU; ++u)
      if (base + 32 * u >= n) x[u] = INFINITY;
    join_kernels(d, x, k.scale, m, acc);
  }
  if (EXTRA && nx > 0) {
    const float x[2] = {l32 < nx ? X[l32] : INFINITY, l32 + 32 < nx ? X[l32 + 32] : INFINITY};
    join_kernels(d, x, k.scale, m, acc);
  }
  const double top = half_max_d(m);
  const double total = half_sum_d(m > -INFINITY ? (double)acc * (double)ex2((float)(m - top)) : 0.0);
  return top + log2_acc((float)total) - k.log_norm;
}

// Update step of one sequence (Section 4.3, last paragraph of Section 4.4; update lines of Algorithm 1)
// by one wavefront, one lane per candidate position (k_max <= 64).  Every lane reads its position's
// distance at once; accepted positions that pass the open-interval filter are appended in position
// order (rank = number of passing positions before it, from a ballot).
// d: the lane's distance (lanes <= r, below kb), H: the draft entropy of the rejected position (lane r).
// Returns the status bits of the step (complete in the lane that finishes the sequence: lane r, or 63);
// with or_status they are also OR-ed into status[b].
struct UpdateIn {
  int nA, nR, ent_cnt;
  double ent_sum;
};
// (by scalar loads, early: the last lane needs them at the very end)
__device__ __forceinline__ UpdateIn update_inputs(const UpdateArgs& a, int b) {
  return UpdateIn{scalar_load(a.nA + b), scalar_load(a.nR + b), scalar_load(a.ent_cnt + b), scalar_load(a.ent_sum + b)};
}
__device__ inline uint32_t update_sequence_core(const UpdateArgs& a, const UpdateIn& in, int b, int lane, int r, int kb, float d,
                                                float H, bool or_status = true) {
  const int nA = in.nA, nR = in.nR;
  double ent_sum = in.ent_sum;
  int ent_cnt = in.ent_cnt;
  if (!(lane <= r && lane < kb)) d = 0.f;
  const bool pass = inside_open_interval(d, a.d_eps);
  uint32_t st = 0;
  // accepted positions 0 .. r-1
  const unsigned long long acc = __ballot(pass && lane < r);
  if (pass && lane < r) {
    const int slot = nA + __popcll(acc & ((1ull << lane) - 1ull));
    if (slot < a.cap) a.LA[(size_t)b * a.cap + slot] = d;
  }
  const int nA_new = min(nA + __popcll(acc), a.cap);
  if (nA + __popcll(acc) > a.cap) st |= ADASD_ST_OVERFLOW;
  // the lane of the rejected position finishes the sequence (with all 64 positions accepted: the last lane)
  const int fin = r < 64 ? r : 63;
  // Running sums of the lists about their first elements: kept from the moment a list reaches kSumsMin
  // samples (added up from scratch in that call), so short lists cost nothing here.
  if (a.mom && (nA_new >= kSumsMin || nR + 1 >= kSumsMin)) {       // (uniform)
    const bool rej_appended = r < kb && __shfl((int)pass, fin) && nR < a.cap;
    const int nR_after = nR + (rej_appended ? 1 : 0);
    const float d_rej = __shfl(d, fin);
    if (nA_new >= kSumsMin && nA_new > nA) {
      const float* LAb = a.LA + (size_t)b * a.cap;
      const double c = (double)LAb[0];          // nA >= kSumsMin - 64 > 0: the first element is an old one
      double s1 = 0.0, s2 = 0.0;
      if (nA < kSumsMin) {                       // the list crosses the mark: everything it held before
        for (int j = lane; j < nA; j += 64) {
          const double e = (double)LAb[j] - c;
          s1 += e;
          s2 += e * e;
        }
      }
      if (pass && lane < r && nA + __popcll(acc & ((1ull << lane) - 1ull)) < a.cap) {
        const double e = (double)d - c;
        s1 += e;
        s2 += e * e;
      }
      s1 = wave_sum_d(s1);
      s2 = wave_sum_d(s2);
      if (lane == 0) {
        const bool fresh = nA < kSumsMin;
        a.mom[4 * b + 0] = (fresh ? 0.0 : a.mom[4 * b + 0]) + s1;
        a.mom[4 * b + 1] = (fresh ? 0.0 : a.mom[4 * b + 1]) + s2;
      }
    }
    if (nR_after >= kSumsMin && rej_appended) {
      const float* LRb = a.LR + (size_t)b * a.cap;
      const double c = (double)LRb[0];
      double s1 = 0.0, s2 = 0.0;
      if (nR < kSumsMin) {
        for (int j = lane; j < nR; j += 64) {
          const double e = (double)LRb[j] - c;
          s1 += e;
          s2 += e * e;
        }
      }
      if (lane == 0) {
        const double e = (double)d_rej - c;
        s1 += e;
        s2 += e * e;
      }
      s1 = wave_sum_d(s1);
      s2 = wave_sum_d(s2);
      if (lane == 0) {
        const bool fresh = nR < kSumsMin;
        a.mom[4 * b + 2] = (fresh ? 0.0 : a.mom[4 * b + 2]) + s1;
        a.mom[4 * b + 3] = (fresh ? 0.0 : a.mom[4 * b + 3]) + s2;
      }
    }
  }
  if (lane != fin) return st;
  int nR_new = nR;
  if (r < kb) {
    if (isfinite(H)) {
      ent_sum += (double)H;
      ent_cnt += 1;
      a.ent_sum[b] = ent_sum;
      a.ent_cnt[b] = ent_cnt;
    }
    if (pass) {
      if (nR < a.cap) a.LR[(size_t)b * a.cap + nR_new++] = d;
      else st |= ADASD_ST_OVERFLOW;
    }
  }
  a.nA[b] = nA_new;
  a.nR[b] = nR_new;
  a.T_G[b] = ent_cnt > 0 ? (float)(ent_sum / (double)ent_cnt) : 0.f;
  if (or_status && a.status && st) a.status[b] |= st;
  return st;
}

// The words of a sequence that its decisions and their update go by, all asked for ahead of everything else, so that they and
// what the positions need are one latency.  The lists' constants and first samples come with them, before it is known how long
// the lists are.  (By scalar loads the lengths were waited for one after the other, in front of everything else.)  Decision kernel (us),
// k = 8, 32 sequences, lists of 64 6.8 -> 5.9, 128 x 16 8.8 -> 8.0, float 8 x 20, lists of 256 8.7 -> 7.8; whole calls,
// decisions in the token kernel: 1 x 4 x 32000 float 13.3 -> 12.9, 1 x 8 x 128256 16.1 -> 15.6.
// (The state is only written once all have read it.)
struct SequenceIn {
  int raw_len, seq, rnd, nA, nR;       // the same in every lane
  int ent_cnt;
  double ent_sum;
};
__device__ __forceinline__ SequenceIn ask_sequence(const DecideArgs& a, const UpdateArgs& upd, int b, bool update) {
  SequenceIn in{a.map.K, b, (int)a.round0, 0, 0, 0, 0.0};
  if (a.nA && a.nR) {
    in.nA = lane_load(a.nA + b);
    in.nR = lane_load(a.nR + b);
  }
  if (a.map.draft_len) in.raw_len = lane_load(a.map.draft_len + b);
  if (a.seq_id) in.seq = (int)lane_load(a.seq_id + b);
  if (a.round) in.rnd = (int)lane_load(a.round + b);
  if (update && upd.B > 0) {
    in.ent_cnt = lane_load(upd.ent_cnt + b);
    in.ent_sum = lane_load(upd.ent_sum + b);
  }
  return in;
}

struct DecideShared {
  float extra[ADASD_MAX_K];         // in-loop appends: this round's distances that pass the filter, in position order
  uint8_t n_before[ADASD_MAX_K];    // in-loop appends: how many of them come from earlier positions
  double mom[kWaves][4];            // per-wave shifted moments of the two lists (long histories)
  double lse2[ADASD_MAX_K][2];      // normalisers of the candidate positions (for the sampling plan)
  uint8_t outcome[ADASD_MAX_K];     // kAccepted, kBroken (non-finite rows), kBadToken; none of them: rejected
  int32_t token[ADASD_MAX_K];       // the drafted tokens
  float dist[ADASD_MAX_K];          // the round's distances (in-loop appends; the fused update step)
  float hq[ADASD_MAX_K];            // the round's draft entropies (the fused update step)
};
constexpr int kAccepted = 1, kBroken = 2, kBadToken = 4;

// Everything a candidate position needs from memory, and its two uniforms.
struct PosLoad {
  int x;
  bool x_ok;
  float zp, zq, p0, p1;
  RowResult rp, rq;
  double log_u1, u2;
};

template <int DT>
__device__ __forceinline__ PosLoad load_position(const DecideArgs& a, const Workspace& ws, int b, int i, uint32_t rnd,
                                                 uint32_t seq) {
  const int l32 = threadIdx.x & 31, K = a.map.K;
  PosLoad L;
  const size_t o = (size_t)b * K + i;
  L.x = a.draft_tokens[o];
  L.x_ok = L.x >= 0 && L.x < a.map.V;
  const char* prow = a.map.base[0] +
      ((int64_t)b * a.map.seq_stride[0] + (int64_t)i * a.map.pos_stride[0]) * Elem<DT>::bytes;
  const char* qrow = a.map.base[1] +
      ((int64_t)b * a.map.seq_stride[1] + (int64_t)i * a.map.pos_stride[1]) * Elem<DT>::bytes;
  if (a.tok) {            // looked up already (by the JS kernel, or by the shard that owns the column)
    const float2 z = a.tok[o];
    L.zp = z.x;
    L.zq = z.y;
  } else {
    L.zp = load_elem<DT>(prow, L.x_ok ? L.x : 0);
    L.zq = load_elem<DT>(qrow, L.x_ok ? L.x : 0);
  }
  L.rp = ws.rows[2 * o];
  L.rq = ws.rows[2 * o + 1];
  L.p0 = L.p1 = 0.f;
  if (a.jsd_split > 0) {
    const float* part = reinterpret_cast<const float*>(ws.part2 + o * kMaxSplit);
    L.p0 = l32 < a.jsd_split ? part[2 * l32] : 0.f;
    L.p1 = l32 + 32 < a.jsd_split ? part[2 * (l32 + 32)] : 0.f;
  }
  const U4 r = philox4x32_10(0u, (uint32_t)i, rnd, seq, a.seed_lo, a.seed_hi);
  // u1 = (w + 0.5) / 2^24 rounded to float: 3e-8 relative, i.e. 3e-8 absolute on its logarithm
  L.log_u1 = kLn2 * log2_acc((float)(((double)(r.w[0] >> 8) + 0.5) * (1.0 / 16777216.0)));
  L.u2 = ((double)(r.w[1] >> 8) + 0.5) * (1.0 / 16777216.0);
  return L;
}

// Two-kernel path: the JS kernel left one partial sum per slice.  Half a wavefront adds them up in a
// fixed tree, corrects the common scale to first order (the weights were formed with the float
// roundings cp, cq of the normalisers, i.e. they are p(1+c), q(1+c') with c = ln2 (lse2_p - cp)) and
// takes the root.
__device__ __forceinline__ float fold_distance(const PosLoad& L) {
  const double A = half_sum_d((double)L.p0 + (double)L.p1);
  const double c0 = kLn2 * (L.rp.lse2 - (double)(float)L.rp.lse2), c1 = kLn2 * (L.rq.lse2 - (double)(float)L.rq.lse2);
  double D = 0.5 * A * (1.0 - 0.5 * (c0 + c1));   // bits
  D = fmin(fmax(D, 0.0), 1.0);
  return (L.rp.bad || L.rq.bad) ? NAN : (float)sqrt(D);
}

// The hand-off words that the single-read statistics kernel left for `count` positions from `first` on go
// back to zero (they are only read inside that kernel, which has finished; the next call finds them clear).
// The stores are dealt to the threads from the last one backwards: the first wavefront, which carries the
// latency chains of these kernels, gets none unless there are more than 192 words.
template <int T>
__device__ __forceinline__ void clear_exchange_words(const DecideArgs& a, const Workspace& ws, size_t first, int count) {
  if (a.xchg_split <= 0) return;
  const int per_pos = a.xchg_split * kXchgWords;
  for (int j = T - 1 - (int)threadIdx.x; j < count * per_pos; j += T) {
    const int i = j / per_pos, w = j - i * per_pos;
    __hip_atomic_store(ws.xchg + (first + i) * (size_t)(kMaxSplit * kXchgWords) + w, 0ull, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  }
}

// The same for the positions of sequence b by the wavefronts of a workgroup but the first.
__device__ __forceinline__ void clear_words_beside(const DecideArgs& a, const Workspace& ws, int b) {
  const int K = a.map.K, per_pos = a.xchg_split * kXchgWords;
  uint64_t* words = ws.xchg + (size_t)b * K * (kMaxSplit * kXchgWords);
  for (int i = 0; i < K; ++i, words += kMaxSplit * kXchgWords)
    for (int w = (int)threadIdx.x - 64; w < per_pos; w += kBlock - 64)
      __hip_atomic_store(words + w, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ double first_lane(double v) {
  return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)), __builtin_amdgcn_readfirstlane(__double2loint(v)));
}

// The round, as decided, applied to the sequence's state by one wavefront.  Returns the status bits (in every lane).
__device__ __forceinline__ uint32_t apply_round(const UpdateArgs& upd, const UpdateIn& before, int b, int r, int kb, const DecideShared& sh) {
  const int lane = threadIdx.x & 63;
  float d = 0.f, H = 0.f;
  if (lane <= r && lane < kb) d = sh.dist[lane];
  if (lane == r && r < kb) H = sh.hq[r];
  const uint32_t st = update_sequence_core(upd, before, b, lane, r, kb, d, H, false);
  return (uint32_t)__builtin_amdgcn_readlane((int)st, r < 64 ? r : 63);
}

// The decisions of one sequence by one workgroup of T threads, LP lanes to a position: with 64 the lower half of the
// wavefront takes the accepted list and the upper half the rejected one, with 32 one list comes after the other.  HIST: the
// lists' constants were formed by the statistics launch; else every group of lanes adds up the lists' moments
// for itself.  Either way nothing but the outcomes goes through shared memory, and nobody waits for anybody before the round
// is decided.  INLOOP: the accepted list grows
// inside the verification loop (Algorithm 1): position i sees the list of the state followed by the
// distances of positions 0..i-1 of this round that pass the open-interval filter, up to the capacity.
// REPLICA: several workgroups decide the same sequence, each for itself.  One of them (`writer`) leaves what is decided,
// and the caller applies the round and leaves the status once all of them have read the state.
struct Decided {        // the same in every lane (REPLICA)
  int r, kb;
  uint32_t st;
  SamplePlan plan;
};
template <int DT, bool INLOOP, bool HIST, int T, int LP, bool REPLICA = false>
__device__ __forceinline__ Decided decide_sequence(const DecideArgs& a, const UpdateArgs& upd, const Workspace& ws, int b,
                                                   const SequenceIn& in, DecideShared& sh, bool writer = true) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, grp = tid / LP;
  const bool lead = (tid & (LP - 1)) == 0;
  constexpr int kGroups = T / LP;
  const int K = a.map.K;

  auto load_pos = [&](int i) { return load_position<DT>(a, ws, b, i, (uint32_t)uniform(in.rnd), (uint32_t)uniform(in.seq)); };
  PosLoad pos;
  // (what stands past the window is asked for as well, but for logits, so that nothing waits for its length)
  if (grp < (a.tok ? K : min(max(uniform(in.raw_len), 0), K))) pos = load_pos(grp);
  const int raw_len = uniform(in.raw_len), kb = min(max(raw_len, 0), K);
  uint32_t st = raw_len != kb ? ADASD_ST_BAD_LENGTH : 0u;
  const int min_n = a.kde_min_n < 2 ? 2 : a.kde_min_n;
  int nA = 0, nR = 0;
  const float* LA = nullptr;
  const float* LR = nullptr;
  if (a.LA && a.LR && a.nA && a.nR) {
    nA = min(max(uniform(in.nA), 0), a.cap);
    nR = min(max(uniform(in.nR), 0), a.cap);
    LA = a.LA + (size_t)b * a.cap;
    LR = a.LR + (size_t)b * a.cap;
  }

  // What the statistics launch left of the lists, and the lists' first samples.  (INLOOP: without the samples.  Their joining, in front
  // of the loop over lists that differ from position to position, cost 16 x 6 x 32003 0.3 us.)
  constexpr int Q = LP == 64 ? 1 : 2;
  const bool upper = LP == 64 && (tid & 32) != 0;
  const bool listed = LA != nullptr && a.cap > 0 && !a.relaxed_off;
  float head[Q][kHalfU] = {};
  Kde k[Q] = {};
  bool ok[Q] = {};
  double c[Q] = {}, s1[Q] = {}, s2[Q] = {};
  if (listed) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const bool rej = upper || q == 1;
      if (HIST) {
        const HistRecord* rec = a.hist + b;
        k[q] = rec->k[rej];
        ok[q] = rec->ok[rej] != 0;
        if (INLOOP) {
          c[q] = rec->c[rej];
          s1[q] = rec->s1[rej];
          s2[q] = rec->s2[rej];
        }
      }
      if (!INLOOP) {
#pragma unroll
        for (int u = 0; u < kHalfU; ++u) head[q][u] = (rej ? LR : LA)[min((tid & 31) + 32 * u, a.cap - 1)];
      }
    }
  }
  int n_room = 0;        // in-loop appends the list can still take
  if (INLOOP) {
    // All distances of the round first: the groups fold them, one wavefront ranks those that pass.
    for (int i = grp; i < kb; i += kGroups) {
      const size_t o = (size_t)b * K + i;
      const PosLoad L = (i == grp) ? pos : load_pos(i);
      float dv;
      if (a.jsd_split > 0) {
        dv = fold_distance(L);
        if (lead && writer) a.d_js[o] = dv;
      } else {
        dv = (L.rp.bad || L.rq.bad) ? NAN : a.d_js[o];
      }
      if (lead) sh.dist[i] = dv;
    }
    __syncthreads();
    if (wave == 0) {
      const float dv = lane < kb ? sh.dist[lane] : NAN;
      const bool pass = inside_open_interval(dv, a.d_eps);
      const unsigned long long mask = __ballot(pass);
      const int rank = __popcll(mask & ((1ull << lane) - 1ull));
      if (lane < kb) sh.n_before[lane] = (uint8_t)rank;
      if (pass) sh.extra[rank] = dv;
    }
    __syncthreads();
    n_room = LA ? max(a.cap - nA, 0) : 0;
  }
  // the Bayesian test needs enough samples in both lists, and spread (else P(A|d) = 0).
  const bool kde_on = kb > 0 && !a.relaxed_off && LA != nullptr && nR >= min_n && (INLOOP ? nA + n_room >= min_n : nA >= min_n);

  // ---- the lists: this lane's (LP = 64), or both
  const float* L[Q];
  int n[Q];
  auto constants = [&](int q, int ne) {
    const bool rej = upper || q == 1;
    double m1 = s1[q], m2 = s2[q];
    if (INLOOP) add_moments(sh.extra, rej ? 0 : ne, c[q], m1, m2);
    ok[q] = kde_constants(m1, m2, rej ? nR : nA + ne, rej ? nA + ne : nR, a.bw_rule, &k[q]);
  };
  if (kde_on) {          // uniform over the workgroup
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const bool rej = upper || q == 1;
      L[q] = rej ? LR : LA;
      n[q] = rej ? nR : nA;
      if (!HIST) {
        c[q] = n[q] > 0 ? (double)L[q][0] : 0.0;
        half_moments(L[q], n[q], c[q], s1[q], s2[q]);
        if (!INLOOP) constants(q, 0);
      }
      if (INLOOP && n[q] == 0) c[q] = (double)sh.extra[0];       // (only used once an extra exists)
    }
  }

  for (int i = grp; i < kb; i += kGroups) {
    if (i != grp) pos = load_pos(i);
    const size_t o = (size_t)b * K + i;
    const RowResult& rp = pos.rp;
    const RowResult& rq = pos.rq;
    const bool bad = rp.bad || rq.bad;
    float dv;
    if (INLOOP) {
      dv = sh.dist[i];
    } else {
      if (a.jsd_split > 0) {
        dv = fold_distance(pos);
        if (lead && writer) a.d_js[o] = dv;
      } else {
        dv = a.d_js[o];
      }
      if (lead) sh.dist[i] = bad ? NAN : dv;
    }
    double PA = 0.0;
    const int ne = INLOOP ? min((int)sh.n_before[i], n_room) : 0;
    if (kde_on && !bad && (!INLOOP || nA + ne >= min_n)) {       // (uniform over the position's lanes)
      double j[2];
      bool both = true;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        if (INLOOP) constants(q, ne);
        j[q] = half_log_joint<INLOOP>((double)dv, L[q], head[q], n[q], sh.extra, upper || q == 1 ? 0 : ne, k[q]);
        both = both && ok[q];
      }
      if (LP == 64) {
        j[1] = j[0];
        swap_halves(j[0], j[1]);
        both = __all(both) != 0;
      }
      if (both) PA = 1.0 / (1.0 + (double)ex2((float)(j[1] - j[0])));
    }
    if (!lead) continue;
    sh.hq[i] = bad ? NAN : rq.H;
    sh.lse2[i][0] = rp.lse2;
    sh.lse2[i][1] = rq.lse2;
    sh.token[i] = pos.x;
    if (bad) {
      if (writer) {
        if (a.H_p) a.H_p[o] = NAN;
        a.H_q[o] = NAN;
        a.d_js[o] = NAN;
        if (a.p_accept) a.p_accept[o] = NAN;
        if (a.accept_mask) a.accept_mask[o] = 0;
      }
      sh.outcome[i] = kBroken;
      continue;
    }
    // speculative-sampling test: accept with probability min(1, p(x)/q(x)), in the log domain; or the
    // loop's own match test: accept with probability p(x)
    int base = 0;
    if (pos.x_ok && a.base_test == 1) {
      base = pos.log_u1 < (double)pos.zp - rp.lse2 * kLn2;
    } else if (pos.x_ok) {
      double lp = (double)pos.zp - rp.lse2 * kLn2;
      double lq = (double)pos.zq - rq.lse2 * kLn2;
      double log_ratio = lp - lq;
      if (log_ratio > 0.0) log_ratio = 0.0;
      base = pos.log_u1 < log_ratio;   // false for NaN (both probabilities zero)
    }
    const int relaxed = a.reject_rule == 1 ? (PA >= 0.5) : (pos.u2 < PA);
    if (writer) {
      if (a.p_accept) a.p_accept[o] = (float)PA;
      if (a.accept_mask) a.accept_mask[o] = (uint8_t)(base | (relaxed << 1));
    }
    sh.outcome[i] = (base || relaxed ? kAccepted : 0) | (pos.x_ok ? 0 : kBadToken);   // rejected only if both tests reject
  }
  for (int i = kb + tid; writer && i < K; i += T) {      // positions past the window
    const size_t o = (size_t)b * K + i;
    if (a.H_p) a.H_p[o] = 0.f;
    a.H_q[o] = 0.f;
    a.d_js[o] = 0.f;
    if (a.p_accept) a.p_accept[o] = 0.f;
    if (a.accept_mask) a.accept_mask[o] = 0;
  }
  __syncthreads();
  if (!REPLICA) clear_exchange_words<T>(a, ws, (size_t)b * K, K);      // (REPLICA: by the caller)
  if (!REPLICA && wave != 0) return {};

  // ---- one wavefront, one lane per position: first rejection, sampling plan, the round applied to the state
  // (the status comes from the outcomes: a word of its own would have to be cleared, with a barrier, before the first position
  // can set a bit of it)
  const int outcome = lane < kb ? sh.outcome[lane] : kAccepted;
  const unsigned long long rejected = __ballot(!(outcome & kAccepted));
  if (__any(outcome & kBroken)) st |= ADASD_ST_NONFINITE;
  if (__any(outcome & kBadToken)) st |= ADASD_ST_BAD_TOKEN;
  const int r = rejected ? __ffsll((long long)rejected) - 1 : kb;
  const auto plan_of = [&](int x, bool valid, double lse2_p, double lse2_q) {
    SamplePlan plan{r, 0, 1, -1, 0.0, 0.0};          // bonus row: Gumbel-max needs no normaliser
    if (r < kb) {
      plan.residual = 1;
      if (a.base_test == 1) {
        // replacement from the target row without the drafted token (a broken token excludes nothing)
        const bool x_ok = x >= 0 && x < a.map.V;
        plan.residual = x_ok ? 2 : 0;
        plan.excluded = x_ok ? x : -1;
      }
      plan.valid = valid;
      plan.lse2_p = lse2_p;
      plan.lse2_q = lse2_q;
    }
    return plan;
  };
  if (!REPLICA) {
    uint32_t st_upd = 0;
    if (upd.B > 0) st_upd = apply_round(upd, UpdateIn{in.nA, in.nR, in.ent_cnt, in.ent_sum}, b, r, kb, sh);      // (the lists were only read above)
    if (lane == 0) {
      a.n_accept[b] = r;
      ws.plan[b] = r < kb ? plan_of(sh.token[r], !(sh.outcome[r] & kBroken), sh.lse2[r][0], sh.lse2[r][1]) : plan_of(-1, true, 0.0, 0.0);
      a.status[b] = st | st_upd;
    }
    return {};
  }
  Decided out{r, kb, st, {}};
  const int at = min(r, ADASD_MAX_K - 1);
  out.plan = plan_of(__builtin_amdgcn_readfirstlane(sh.token[at]), !(__builtin_amdgcn_readfirstlane((int)sh.outcome[at]) & kBroken),
                     first_lane(sh.lse2[at][0]), first_lane(sh.lse2[at][1]));
  if (writer && tid == 0) a.n_accept[b] = r;
  return out;
}

}  // namespace adasd

namespace adasd {

__device__ inline void update_sequence(const UpdateArgs& a, int b, int lane, int r, int kb) {
  float d = 0.f, H = 0.f;
  if (lane <= r && lane < kb) d = a.d_js[(size_t)b * a.K + lane];
  if (lane == r && r < kb) H = a.H_q[(size_t)b * a.K + r];
  update_sequence_core(a, update_inputs(a, b), b, lane, r, kb, d, H);
}


// ---------------------------------------------------------------------------------------------
// Long histories.  The cost of the Bayesian test grows with the lists (Section 4.4 flags it): with
// thousands of samples per list one workgroup per sequence and half a wavefront per position is far
// too little.  Here one workgroup of 256 threads takes ONE position: every thread walks a stride of
// both lists once (running reference and rescaled sum, so no separate pass for the maximum), the
// workgroups of a sequence leave one record per position, and the one that arrives last takes the
// sequence's decisions (first rejection, sampling plan, status, update step).
// With few workgroups this is a chain of latencies, with many the double-precision arithmetic of the samples counts, and the
// wavefronts in flight: samples are walked in groups of four per thread, as many groups as the longer list fills (all 16 at
// once took 143 registers and did four times the work for a list of a thousand), and the two lists' groups side by side.
// Kernel (us), all 16 / groups: 32 x 8 positions, lists of 1024 8.9 / 7.7, 128 x 16 23.8 / 15.4, 128 x 40 51.2 / 29.7,
// 64 x 16 ragged, lists of 4096 15.7 / 13.8.
// ---------------------------------------------------------------------------------------------
struct WideShared {
  double m[2][kWaves], s[2][kWaves];
  int last;
  int n_pass;           // in-loop appends: earlier positions of this round that pass the filter
};

constexpr int kWideU = 16;   // samples per thread in flight: one workgroup walks a list alone, so the latency of
                             // a load is only hidden by the thread's own other loads

// A thread's samples of a list, from `first` on in steps of the workgroup: asked for and joined in groups of kWideG, as many as
// the list fills (`first` less the thread's own index is uniform).
constexpr int kWideG = 4;
__device__ __forceinline__ void ask_terms(const float* L, int first, int n, float (&x)[kWideU / kWideG][kWideG]) {
  const int start = first - (int)threadIdx.x;
#pragma unroll
  for (int g = 0; g < kWideU / kWideG; ++g) {
    if (start + g * kWideG * kBlock >= n) break;
#pragma unroll
    for (int u = 0; u < kWideG; ++u) x[g][u] = L[min(first + (g * kWideG + u) * kBlock, n - 1)];
  }
}
__device__ __forceinline__ void join_group(double d, float (&x)[kWideG], int g, int first, int n, double scale, double& m, double& s) {
#pragma unroll
  for (int u = 0; u < kWideG; ++u)
    if (first + (g * kWideG + u) * kBlock >= n) x[u] = INFINITY;
  join_kernels(d, x, scale, m, s);
}

// Workgroup-wide log-sum of N lists' per-thread (m, s) pairs at once: common maximum, rescaled sums (a
// thread without samples has s = 0).  out[q] = log2 of the sum of list q.
template <int N>
__device__ __forceinline__ void joint_reduce(const double (&m)[N], const double (&s)[N], WideShared& w, double (&out)[N]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double M[N], sc[N];
#pragma unroll
  for (int q = 0; q < N; ++q) {
    M[q] = half_max_d(m[q]);
    double other = M[q];
    swap_halves(M[q], other);
    M[q] = fmax(M[q], other);
    sc[q] = m[q] > -INFINITY ? s[q] * (double)ex2((float)(m[q] - M[q])) : 0.0;
    sc[q] = wave_sum_d(sc[q]);
  }
  __syncthreads();
  if (lane == 0) {
#pragma unroll
    for (int q = 0; q < N; ++q) {
      w.m[q][wave] = M[q];
      w.s[q][wave] = sc[q];
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < N; ++q) {
    double Mb = w.m[q][0];
#pragma unroll
    for (int v = 1; v < kWaves; ++v) Mb = fmax(Mb, w.m[q][v]);
    double total = 0.0;
#pragma unroll
    for (int v = 0; v < kWaves; ++v)
      total += w.m[q][v] > -INFINITY ? w.s[q][v] * (double)ex2((float)(w.m[q][v] - Mb)) : 0.0;
    out[q] = Mb + log2_acc((float)total);
  }
}

// A list of any length, streamed.
__device__ inline void stream_terms(double d, const float* L, int n, double scale, double& m, double& s) {
#pragma unroll 1
  for (int first = threadIdx.x; first - (int)threadIdx.x < n; first += kWideU * kBlock) {
    float x[kWideU / kWideG][kWideG];
    ask_terms(L, first, n, x);
#pragma unroll
    for (int g = 0; g < kWideU / kWideG; ++g) join_group(d, x[g], g, first, n, scale, m, s);
  }
}

// Sums of x - c and of its square over a group of a thread's samples.
__device__ __forceinline__ void group_moments(const float (&x)[kWideG], int g, int first, int n, double c, double& s1, double& s2) {
#pragma unroll
  for (int u = 0; u < kWideG; ++u) {
    const double e = first + (g * kWideG + u) * kBlock < n ? (double)x[u] - c : 0.0;
    s1 += e;
    s2 += e * e;
  }
}

// The same over the two lists, by the workgroup (where no earlier kernel left them): from the registers that hold the lists
// (`resident`; a second read of them cost a round of 128 x 16 positions 2 to 4 us of 70), or streamed.
__device__ inline void list_moments(const DecideArgs& a, int b, const float* LA, const float* LR, int nA, int nR, bool resident,
                                    const float (&xa)[kWideU / kWideG][kWideG], const float (&xr)[kWideU / kWideG][kWideG],
                                    const double (&c)[2], DecideShared& sh, double (&m)[4]) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float* L[2] = {LA, LR};
  const int n[2] = {nA, nR};
  m[0] = m[1] = m[2] = m[3] = 0.0;
  if (resident) {
#pragma unroll
    for (int g = 0; g < kWideU / kWideG; ++g) {
      if (g * kWideG * kBlock >= max(nA, nR)) break;
      group_moments(xa[g], g, tid, nA, c[0], m[0], m[1]);
      group_moments(xr[g], g, tid, nR, c[1], m[2], m[3]);
    }
  } else {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (a.mom && n[q] > kSumsMin) continue;
#pragma unroll 1
      for (int first = tid; first - tid < n[q]; first += kWideU * kBlock) {
        float x[kWideU / kWideG][kWideG];
        ask_terms(L[q], first, n[q], x);
#pragma unroll
        for (int g = 0; g < kWideU / kWideG; ++g) group_moments(x[g], g, first, n[q], c[q], m[2 * q], m[2 * q + 1]);
      }
    }
  }
#pragma unroll
  for (int x = 0; x < 4; ++x) m[x] = wave_sum_d(m[x]);
  if (lane == 0) {
#pragma unroll
    for (int x = 0; x < 4; ++x) sh.mom[wave][x] = m[x];
  }
  __syncthreads();
#pragma unroll
  for (int x = 0; x < 4; ++x)
    m[x] = a.mom && n[x >> 1] > kSumsMin ? a.mom[4 * b + x] : (sh.mom[0][x] + sh.mom[1][x]) + (sh.mom[2][x] + sh.mom[3][x]);
}

template <int DT, bool INLOOP, bool HIST>
__device__ void decide_position_wide(const DecideArgs& a, const UpdateArgs& upd, const Workspace& ws,
                                     PosRecord* records, int b, int i, DecideShared& sh, WideShared& wsh) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = tid & 31, grp = tid >> 5;
  constexpr int kGroups = kBlock / 32;
  const int K = a.map.K;
  constexpr int U = kWideU;
  int kb = K;
  uint32_t st_seq = 0;
  if (a.map.draft_len) {
    const int raw = scalar_load(a.map.draft_len + b);
    kb = min(max(raw, 0), K);
    if (raw != kb) st_seq |= ADASD_ST_BAD_LENGTH;
  }
  const uint32_t seq = a.seq_id ? scalar_load(a.seq_id + b) : (uint32_t)b;
  const uint32_t rnd = a.round ? scalar_load(a.round + b) : a.round0;
  const int nA = min(max(scalar_load(a.nA + b), 0), a.cap), nR = min(max(scalar_load(a.nR + b), 0), a.cap);
  const float* LA = a.LA + (size_t)b * a.cap;
  const float* LR = a.LR + (size_t)b * a.cap;
  const size_t o = (size_t)b * K + i;

  PosRecord rec{0, 0u, 0.f, 0.f};
  HistRecord hist;
  // Lists that were short when the statistics ran have been taken past the line by the round itself: the sequence is done.
  const auto applied_already = [&] { return HIST && max(hist.n[0], hist.n[1]) < kWideMin; };
  if (i >= kb) {
    if (HIST) hist = a.hist[b];
    if (applied_already()) return;
    if (tid == 0) {
      if (a.H_p) a.H_p[o] = 0.f;
      a.H_q[o] = 0.f;
      a.d_js[o] = 0.f;
      if (a.p_accept) a.p_accept[o] = 0.f;
      if (a.accept_mask) a.accept_mask[o] = 0;
    }
  } else {
    // Lists of up to U samples per thread are read ONCE, both at the same time and ahead of everything else, and stay in
    // registers; longer ones are streamed.
    const bool resident = nA <= U * kBlock && nR <= U * kBlock;
    float xa[U / kWideG][kWideG], xr[U / kWideG][kWideG];
    if (resident) {
      ask_terms(LA, tid, nA, xa);
      ask_terms(LR, tid, nR, xr);
    }
    if (HIST) hist = a.hist[b];
    const PosLoad L = load_position<DT>(a, ws, b, i, rnd, seq);
    if (applied_already()) return;       // (here, where the constants are waited for: at the top it was a miss of its own)
    const bool bad = L.rp.bad || L.rq.bad;
    const int min_n = a.kde_min_n < 2 ? 2 : a.kde_min_n;
    int ne = 0;                            // in-loop appends this position sees
    if (INLOOP) {
      // distances of the earlier positions (each workgroup of the sequence forms them for itself)
      for (int j = grp; j < i; j += kGroups) {
        const PosLoad Lj = load_position<DT>(a, ws, b, j, rnd, seq);
        float dv;
        if (a.jsd_split > 0) dv = fold_distance(Lj);
        else dv = (Lj.rp.bad || Lj.rq.bad) ? NAN : a.d_js[(size_t)b * K + j];
        if (l32 == 0) sh.dist[j] = dv;
      }
      __syncthreads();
      if (wave == 0) {
        const float dv = lane < i ? sh.dist[lane] : NAN;
        const bool pass = inside_open_interval(dv, a.d_eps);
        const unsigned long long mask = __ballot(pass);
        if (pass) sh.extra[__popcll(mask & ((1ull << lane) - 1ull))] = dv;
        if (lane == 0) wsh.n_pass = __popcll(mask);
      }
      __syncthreads();
      ne = min(wsh.n_pass, a.cap - nA);
    }
    float d_out;
    if (a.jsd_split > 0) {
      d_out = fold_distance(L);
      if (tid == 0) a.d_js[o] = d_out;
    } else {
      d_out = bad ? NAN : a.d_js[o];
    }
    const double d = (double)d_out;
    const int n_i = nA + ne;
    double PA = 0.0;
    bool reduced = false;
    if (!bad && n_i >= min_n && nR >= min_n) {      // uniform over the workgroup
      Kde kA, kR;
      bool ok;
      if (HIST && ne == 0) {
        kA = hist.k[0];
        kR = hist.k[1];
        ok = hist.ok[0] && hist.ok[1];
      } else {
        const double c[2] = {nA == 0 ? (double)sh.extra[0] : HIST ? hist.c[0] : (double)LA[0], HIST ? hist.c[1] : (double)LR[0]};
        double m[4];
        if (HIST) {
          m[0] = hist.s1[0];
          m[1] = hist.s2[0];
          m[2] = hist.s1[1];
          m[3] = hist.s2[1];
        } else {
          list_moments(a, b, LA, LR, nA, nR, resident, xa, xr, c, sh, m);
        }
        if (INLOOP) add_moments(sh.extra, ne, c[0], m[0], m[1]);
        ok = kde_constants(m[0], m[1], n_i, nR, a.bw_rule, &kA) && kde_constants(m[2], m[3], nR, n_i, a.bw_rule, &kR);
      }
      if (ok) {                      // uniform over the workgroup
        double mm[2] = {-INFINITY, -INFINITY}, ss[2] = {0.0, 0.0}, out[2];
        if (resident) {
          // the two lists side by side: each group is a chain of dependent instructions
#pragma unroll
          for (int g = 0; g < U / kWideG; ++g) {
            if (g * kWideG * kBlock >= max(nA, nR)) break;
            join_group(d, xa[g], g, tid, nA, kA.scale, mm[0], ss[0]);
            join_group(d, xr[g], g, tid, nR, kR.scale, mm[1], ss[1]);
          }
        } else {
          stream_terms(d, LA, nA, kA.scale, mm[0], ss[0]);
          stream_terms(d, LR, nR, kR.scale, mm[1], ss[1]);
        }
        if (INLOOP && tid < ne) {    // the list goes on with the appends
          const float x[1] = {sh.extra[tid]};
          join_kernels(d, x, kA.scale, mm[0], ss[0]);
        }
        joint_reduce<2>(mm, ss, wsh, out);
        reduced = true;
        const double ja = out[0] - kA.log_norm, jr = out[1] - kR.log_norm;
        PA = 1.0 / (1.0 + (double)ex2((float)(jr - ja)));
      }
    }
    // Once all workgroups of the sequence have arrived, the last one changes the state: what a wavefront reads of it (lengths,
    // running sums) and goes by, it has to have read before this one arrives.  joint_reduce has barriers; else one here.
    if (!reduced) __syncthreads();
    if (tid == 0) {
      rec.d = d_out;
      if (bad) {
        if (a.H_p) a.H_p[o] = NAN;
        a.H_q[o] = NAN;
        a.d_js[o] = NAN;
        if (a.p_accept) a.p_accept[o] = NAN;
        if (a.accept_mask) a.accept_mask[o] = 0;
        rec.bits = 2;
        rec.status = ADASD_ST_NONFINITE;
        rec.d = NAN;
      } else {
        int base = 0;
        if (!L.x_ok) {
          rec.status |= ADASD_ST_BAD_TOKEN;
        } else if (a.base_test == 1) {
          base = L.log_u1 < (double)L.zp - L.rp.lse2 * kLn2;
        } else {
          double log_ratio = ((double)L.zp - L.rp.lse2 * kLn2) - ((double)L.zq - L.rq.lse2 * kLn2);
          if (log_ratio > 0.0) log_ratio = 0.0;
          base = L.log_u1 < log_ratio;
        }
        const int relaxed = a.reject_rule == 1 ? (PA >= 0.5) : (L.u2 < PA);
        if (a.p_accept) a.p_accept[o] = (float)PA;
        if (a.accept_mask) a.accept_mask[o] = (uint8_t)(base | (relaxed << 1));
        rec.bits = (base || relaxed) ? 1 : 0;
      }
    }
  }
  // ---- the position's record, then the arrival counter of the sequence
  if (tid == 0) {
    PosRecord* dst = records + o;
    st_agent(&dst->bits, rec.bits);
    st_agent(reinterpret_cast<int*>(&dst->status), (int)rec.status);
    st_agent(&dst->d, rec.d);
    publish_barrier();
    const int ticket = atomicAdd(&ws.ticket2[b * ticket_stride(a.map.B, kTicket2Len)], 1);
    wsh.last = ticket == K - 1;
  }
  __syncthreads();
  clear_exchange_words<kBlock>(a, ws, o, 1);
  if (!wsh.last || wave != 0) return;

  // ---- last workgroup of the sequence, one wavefront, one lane per position
  UpdateIn before{};
  if (upd.B > 0) before = update_inputs(upd, b);
  // Every lane also asks for what the sampling plan and the update step need of ITS position (the
  // normalisers, the drafted token, the draft entropy: all left by earlier kernels), so that nothing is
  // loaded once the rejected position is known; its lane hands them over.
  int bits = 0;
  uint32_t pst = 0;
  float dl = 0.f, Hl = 0.f;
  double lse_p = 0.0, lse_q = 0.0;
  int xl = -1;
  if (lane < K) {
    const size_t ol = (size_t)b * K + lane;
    const PosRecord* src = records + ol;
    bits = ld_agent(&src->bits);
    pst = (uint32_t)ld_agent(reinterpret_cast<const int*>(&src->status));
    dl = ld_agent(&src->d);
    if (lane < kb) {
      lse_p = ws.rows[2 * ol].lse2;
      lse_q = ws.rows[2 * ol + 1].lse2;
      if (a.base_test == 1) xl = a.draft_tokens[ol];
      if (upd.B > 0) Hl = upd.H_q[ol];
    }
  }
  const unsigned long long rejected = __ballot(lane < kb && !(bits & 1));
  const int r = rejected ? __ffsll((long long)rejected) - 1 : kb;
  uint32_t st_all = pst;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) st_all |= __shfl_xor(st_all, off);
  const int src_lane = r < 64 ? r : 63;
  const int bad_r = __shfl(bits, src_lane) & 2;
  const double lse_p_r = __shfl(lse_p, src_lane), lse_q_r = __shfl(lse_q, src_lane);
  const int x_r = __shfl(xl, src_lane);
  if (lane == 0) {
    a.n_accept[b] = r;
    SamplePlan plan;
    plan.row = r;
    plan.excluded = -1;
    if (r < kb) {
      plan.residual = 1;
      if (a.base_test == 1) {
        const bool x_ok = x_r >= 0 && x_r < a.map.V;
        plan.residual = x_ok ? 2 : 0;
        plan.excluded = x_ok ? x_r : -1;
      }
      plan.valid = !bad_r;
      plan.lse2_p = lse_p_r;
      plan.lse2_q = lse_q_r;
    } else {
      plan.residual = 0;
      plan.valid = 1;
      plan.lse2_p = 0.0;
      plan.lse2_q = 0.0;
    }
    ws.plan[b] = plan;
    __hip_atomic_store(&ws.ticket2[b * ticket_stride(a.map.B, kTicket2Len)], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  uint32_t st_upd = 0;
  if (upd.B > 0) {
    // (a position with non-finite rows records nothing, whatever its entropy word holds by now)
    const float H = (lane == r && r < kb && !(bits & 2)) ? Hl : NAN;
    st_upd = update_sequence_core(upd, before, b, lane, r, kb, dl, H, false);
  }
  // one store of the sequence's status word, the update step's bits included (they are complete in its last lane)
  st_upd = __shfl(st_upd, src_lane);
  if (lane == 0) a.status[b] = st_seq | st_all | st_upd;
}

}  // namespace adasd
