// Correction / bonus token (Section 2.1.3: re-sampling from the adjusted distribution; last lines of
// the verification step of Algorithm 1): Gumbel-max over the vocabulary with counter-based Philox
// noise, argmax_v ln w_v - ln(-ln u_v), lowest index on ties.
//
// Fast path: float keys in the log2 domain that are UPPER BOUNDS of the true keys, running top-2 per
// slice and sequence.  The winner is final only if its lower bound beats the runner-up's upper bound.
// Otherwise the workgroup that folds the slices settles the sequence in float64: first among the few
// elements whose upper bound reaches the winner's lower bound (found from the per-slice records, a
// slice with two such elements is scanned again), and only if that is still too close to call, or the
// winner's mass is not certain, over the whole row (exact path).
#include "decide_device.h"
#include "sample_device.h"

namespace adasd {

namespace {

using namespace sampling;

// The scan of a sequence's row(s) under its plan.
template <int DT, bool LONG, bool PRUNE>
__device__ __forceinline__ void scan_plan(const SamplePlan& plan, const char* prow, const char* qrow, int V, int v0, int v1,
                                          int col0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0, uint32_t k1,
                                          Top2& best, Floors& sh, bool& poison) {
  const float cp = (float)plan.lse2_p, cq = (float)plan.lse2_q;
  const PhiloxRow noise = philox_row(c1, c2, c3, k0, k1);
  if (LONG) {
    if (plan.residual == kResidual) scan_long_slice<DT, kResidual, PRUNE>(prow, qrow, V, v0, v1, cp, cq, -1, noise, best, sh, poison);
    else if (plan.residual == kExclude) scan_long_slice<DT, kExclude, PRUNE>(prow, qrow, V, v0, v1, cp, cq, plan.excluded, noise, best, sh, poison);
    else scan_long_slice<DT, kPlain, PRUNE>(prow, qrow, V, v0, v1, cp, cq, -1, noise, best, sh, poison);
    return;
  }
  if (plan.residual == kResidual) scan_slice<DT, kResidual, PRUNE>(prow, qrow, V, v0, v1, cp, cq, -1, col0, noise, best, sh, poison);
  else if (plan.residual == kExclude) scan_slice<DT, kExclude, PRUNE>(prow, qrow, V, v0, v1, cp, cq, plan.excluded, col0, noise, best, sh, poison);
  else scan_slice<DT, kPlain, PRUNE>(prow, qrow, V, v0, v1, cp, cq, -1, col0, noise, best, sh, poison);
}

// Where a sequence's slices leave their words (instead of PlainWords) while those of the statistics kernel are being cleared:
// in the slots of its positions that that kernel does not use (free_slots of them per position, at least half of
// them: a sequence's slices take those of two positions at most).
struct FreeWords {
  uint64_t* base;      // the first free slot of the sequence's first position
  int free_slots;
  __device__ __forceinline__ uint64_t* at(int s) const {
    return base + (s < free_slots ? s : s - free_slots + kMaxSplit) * kXchgWords;
  }
};

__device__ __forceinline__ FreeWords free_words(const DecideArgs& d, const Workspace& ws, int b) {
  return FreeWords{ws.xchg + ((size_t)b * d.map.K * kMaxSplit + d.xchg_split) * kXchgWords, kMaxSplit - d.xchg_split};
}

// What the token kernel does beside the draw: nothing, or (MERGED) the round is still to be applied and the status word to be
// left, by the workgroup that folds the slices.
struct DrawOnly {
  static constexpr bool kMerged = false;
  __device__ __forceinline__ void beside() {}
  __device__ __forceinline__ void ask() {}
  __device__ __forceinline__ uint32_t finish() { return 0u; }
};
struct DrawAndApply {
  static constexpr bool kMerged = true;
  const DecideArgs& d;
  const UpdateArgs& upd;
  const Workspace& ws;
  const DecideShared& sh;
  const Decided& dec;
  int b;
  UpdateIn before;
  // (not before the record is under way: the first workgroup's would be the one that the others' wait for, 0.8 us with 8
  // positions of 32 slices)
  __device__ __forceinline__ void beside() {
    if (blockIdx.x == 0) clear_words_beside(d, ws, b);
  }
  __device__ __forceinline__ void ask() {
    if (upd.B > 0) before = update_inputs(upd, b);
  }
  __device__ __forceinline__ uint32_t finish() { return dec.st | (upd.B > 0 ? apply_round(upd, before, b, dec.r, dec.kb, sh) : 0u); }
};

// The token of sequence b, slice s of S, by one workgroup of kBlock threads.
// Who folds the slices' records: see few_rows.  With that, without the tie loop for wavefronts that have no logit, with the best's
// logits asked for before the folds and the wavefronts folded by every lane for itself, whole calls (us): 1 x 4 x 32000 float 15.79
// -> 14.17, 1 x 8 x 128256 bf16 17.23 -> 16.18, 16 x 6 x 32003 literal 20.35 -> 19.31; 32 x 8 x 128256 the same within noise.  (That
// a last slice can give a sequence up takes up to 0.1 of it back.)
// LONG: a row of more slices than there are hand-off words (see token_split).  The records then go through part3, and have
// landed before the ticket is taken; and a compute unit holds no more than one such workgroup of a few sequences.
template <int DT, bool LONG, bool PRUNE, class Words, class Round>
__device__ __forceinline__ void draw_token(const SampleArgs& a, int S, int chunk, const Workspace& ws, const SamplePlan& plan, uint32_t c2,
                                           uint32_t c3, const Words& slots, Round& round) {
  const int b = blockIdx.y, s = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int V = a.map.V;
  const char* prow = a.map.base[0] + ((int64_t)b * a.map.seq_stride[0] +
                                      (int64_t)plan.row * a.map.pos_stride[0]) * Elem<DT>::bytes;
  const char* qrow = a.map.base[1] + ((int64_t)b * a.map.seq_stride[1] +
                                      (int64_t)plan.row * a.map.pos_stride[1]) * Elem<DT>::bytes;
  const uint32_t c1 = (uint32_t)plan.row | (1u << 16);

  const int nv = vectors_of<DT>(V), v0 = min(s * chunk, nv), v1 = min(v0 + chunk, nv);
  Top2 best{-INFINITY, -1, -INFINITY, -1};
  bool poison = false;
  __shared__ Floors sh_floors;
  if (PRUNE) floors_init(sh_floors);
  scan_plan<DT, LONG, PRUNE>(plan, prow, qrow, V, v0, v1, 0, c1, c2, c3, a.seed_lo, a.seed_hi, best, sh_floors, poison);

  __shared__ Top2 sh_top[kWaves];
  __shared__ float2 sh_logits[kWaves];
  // modes: 0 another workgroup folds; 1 final; 2 settle among the close candidates; 3 broken bonus row; 4 whole row in float64
  __shared__ int sh_mode;
  __shared__ uint32_t sh_status;              // (MERGED) what the status word holds so far
  __shared__ float sh_tau;
  __shared__ double sh_red[kWaves];
  // (residual) the logits of the best element, which the error of its key depends on: every lane asks for its own best's, so
  // that they arrive while the wavefront looks for its best
  const int own = best.i1;
  const bool residual = plan.residual == kResidual;
  float zp = 0.f, zq = 0.f;
  if (!LONG && residual && own >= 0) {
    zp = load_elem<DT>(prow, own);
    zq = load_elem<DT>(qrow, own);
  }
  best = top2_wave_reduce(best);
  best.i2 = __any(poison) ? -2 : -1;          // (the poison marker travels in the runner-up's index)
  if (lane == 0) sh_top[wave] = best;
  if (own == best.i1 && own >= 0) sh_logits[wave] = make_float2(zp, zq);     // (one lane)
  __syncthreads();
  if (wave == 0) {
    // the slice's record: best key and its index, runner-up key, the logits of the best
    const Top2 t0 = sh_top[0], t1 = sh_top[1], t2 = sh_top[2], t3 = sh_top[3];
    static_assert(kWaves == 4, "four wavefronts");
    poison = t0.i2 == -2 || t1.i2 == -2 || t2.i2 == -2 || t3.i2 == -2;
    best = top2_merge(top2_merge(t0, t1), top2_merge(t2, t3));
    const float2 z = sh_logits[best.i1 == t0.i1 ? 0 : best.i1 == t1.i1 ? 1 : best.i1 == t2.i1 ? 2 : 3];
    zp = best.i1 >= 0 ? z.x : 0.f;
    zq = best.i1 >= 0 ? z.y : 0.f;
    bool last = true, arrived = true;
    uint64_t w[kXchgWords];
    const Arrivals arrivals{ws.ticket3, kTicket3Len, b, a.map.B};
    if (LONG) {
      if (lane == 0) {
        Top2* dst = &ws.part3[(size_t)b * kMaxSampleSplit + s];
        st_agent(&dst->k1, best.k1);
        st_agent(&dst->i1, best.i1);
        st_agent(&dst->k2, best.k2);
        st_agent(&dst->i2, poison ? -2 : -1);
      }
      publish_barrier();
      int32_t* count = &ws.ticket3[b * ticket_stride(a.map.B, kTicket3Len)];
      last = last_to_add(add_arrival(count), S);
      if (last) {
        set_arrival(count, 0);
        round.ask();
      }
    } else if (S > 1) {
      pack_draw(DrawRecord{best.k1, best.k2, zp, zq, best.i1, poison}, w);
      last = hand_off(slots, s, S, arrivals, a.wait, [&] { round.ask(); }, w, arrived);
    } else {
      round.ask();
    }
    int mode = 0;
    if (last) {
      // ---- the S records of this sequence folded
      Top2 t{-INFINITY, -1, -INFINITY, -1};
      if (LONG) {
        poison = false;
        for (int j = lane; j < S; j += 64) {
          const Top2* src = &ws.part3[(size_t)b * kMaxSampleSplit + j];
          t = top2_merge(t, Top2{ld_agent(&src->k1), ld_agent(&src->i1), ld_agent(&src->k2), -1});
          poison |= ld_agent(&src->i2) == -2;
        }
        poison = __any(poison);
      } else if (S > 1) {
        if (lane < S) {
          const DrawRecord r = unpack_draw(w);
          t = Top2{r.k1, r.i1, r.k2, -1};
          poison = r.poison;
          zp = r.zp;
          zq = r.zq;
        } else {
          poison = false;
        }
        poison = __any(poison);
      } else if (lane == 0) {
        t = best;
      }
      const Top2 top = top2_wave_reduce(t);
      float margin = kGuard;
      mode = 1;
      if (!arrived) {
        mode = 4;   // (the float64 path looks at every logit, also for broken ones)
      } else if (poison) {
        mode = 3;   // NaN / +inf in the bonus row
      } else if (top.i1 < 0) {
        mode = 4;   // nothing had (certain) mass
      } else {
        if (residual) {
          const int owner = S > 1 ? __ffsll((long long)__ballot(t.i1 == top.i1)) - 1 : 0;
          if (LONG) {
            zp = load_elem<DT>(prow, top.i1);
            zq = load_elem<DT>(qrow, top.i1);
          }
          const float p = ex2(fmaf(lane_value(zp, owner), kLog2e, -(float)plan.lse2_p));
          const float q = ex2(fmaf(lane_value(zq, owner), kLog2e, -(float)plan.lse2_q));
          const float err = kErrRel * (p + q), w = p - q;
          // true key >= key_ub - log2((w+err)/(w-err)); for err/w < 1/2 that is < 3 log2(e) err/w
          if (!(w > 2.f * err)) mode = 4;
          else margin += 3.f * kLog2e * err / w;
        }
        // an element whose upper bound stays below the winner's lower bound cannot be the true winner
        if (mode == 1 && !(top.k1 - top.k2 > margin)) mode = 2;
      }
      if (!LONG && mode == 2 && lane < S) {   // the slices' records, for the search for close candidates
        Top2* dst = &ws.part3[(size_t)b * kMaxSampleSplit + lane];
        st_agent(&dst->k1, t.k1);
        st_agent(&dst->i1, t.i1);
        st_agent(&dst->k2, t.k2);
        publish_barrier();
      }
      if (mode == 1 && lane == 0) a.next_token[b] = top.i1;
      if (lane == 0) sh_tau = top.k1 - margin;
      if (Round::kMerged) {
        const uint32_t st = round.finish();
        if (lane == 0) {
          sh_status = st;
          if (mode == 1) a.status[b] = st;
        }
      }
    }
    if (lane == 0) sh_mode = mode;
  } else {
    round.beside();
  }
  __syncthreads();
  const int mode = sh_mode;
  if (mode <= 1) return;
  if (mode == 3) {
    if (tid == 0) {
      a.next_token[b] = -1;
      a.status[b] = (Round::kMerged ? sh_status : a.status[b]) | ADASD_ST_NONFINITE;
    }
    return;
  }
  uint32_t bits = ADASD_ST_EXACT_PATH;
  const int excluded = plan.residual == kExclude ? plan.excluded : -1;
  int tok = -1;
  if (mode == 2) {
    __shared__ RefineShared sh_refine;
    tok = sample_refine<DT>(prow, qrow, plan.residual, excluded, V, b, S, sh_tau, (float)plan.lse2_p, (float)plan.lse2_q, plan.lse2_p,
                            plan.lse2_q, c1, c2, c3, a.seed_lo, a.seed_hi, ws, sh_red, sh_refine);
  }
  if (tok < 0)
    tok = sample_exact<DT>(prow, qrow, plan.residual == kResidual, excluded, V, c1, c2, c3, a.seed_lo,
                           a.seed_hi, sh_red, &bits);
  if (tid == 0) {
    a.next_token[b] = tok;
    a.status[b] = (Round::kMerged ? sh_status : a.status[b]) | bits;
  }
}

template <int DT, bool LONG, bool PRUNE>
__global__ void __launch_bounds__(kBlock, LONG ? 4 : 7) k_sample(SampleArgs a, int S, int chunk, Workspace ws) {
  warm_kernargs<sizeof(SampleArgs) + 2 * sizeof(int) + sizeof(Workspace)>();
  const int b = blockIdx.y;
  // (by scalar loads, all at once: the kernel before this one has left them)
  const SamplePlan plan = scalar_load(ws.plan + b);
  const uint32_t c2 = a.round ? scalar_load(a.round + b) : a.round0;
  const uint32_t c3 = a.seq_id ? scalar_load(a.seq_id + b) : (uint32_t)b;
  if (!plan.valid) {
    if (blockIdx.x == 0 && threadIdx.x == 0) a.next_token[b] = -1;   // status already carries NONFINITE
    return;
  }
  DrawOnly round;
  draw_token<DT, LONG, PRUNE>(a, S, chunk, ws, plan, c2, c3, PlainWords{ws.xchg + (size_t)b * kMaxSplit * kXchgWords}, round);
}

// Decisions and token in one launch, for rounds of so few positions and slices that deciding a sequence in every
// workgroup of its token scan costs less than a launch: the first one leaves what is decided, and the one that
// folds the slices applies the round, when all have read the state.  One turn of the positions: a wavefront to each of up
// to four, half a wavefront to each of up to eight.
template <int DT, bool INLOOP, int LP, bool PRUNE>
__global__ void __launch_bounds__(kBlock, 4) k_decide_sample(DecideArgs d, UpdateArgs upd, SampleArgs a, int S, int chunk, Workspace ws) {
  warm_kernargs<sizeof(DecideArgs) + sizeof(UpdateArgs) + sizeof(SampleArgs) + 2 * sizeof(int) + sizeof(Workspace)>();
  __shared__ DecideShared sh;
  const int b = blockIdx.y;
  const SequenceIn in = ask_sequence(d, upd, b, false);
  const Decided dec = decide_sequence<DT, INLOOP, true, kBlock, LP, true>(d, upd, ws, b, in, sh, blockIdx.x == 0);
  DrawAndApply round{d, upd, ws, sh, dec, b, {}};
  if (!dec.plan.valid) {          // (uniform over the sequence's workgroups)
    if (threadIdx.x >= 64) {
      round.beside();
      return;
    }
    if (S > 1) {                  // (records without a content: once all have been sent, the state has been read)
      const uint64_t none = record_word(1u, 0.f);
      uint64_t w[kXchgWords] = {none, none, none};
      bool arrived;               // (sent is enough)
      if (!hand_off(free_words(d, ws, b), blockIdx.x, S, Arrivals{ws.ticket3, kTicket3Len, b, a.map.B}, a.wait, [&] { round.ask(); }, w,
                    arrived))
        return;
    } else {
      round.ask();
    }
    const uint32_t st = round.finish();
    if (threadIdx.x == 0) {
      a.next_token[b] = -1;
      a.status[b] = st;
    }
    return;
  }
  draw_token<DT, false, PRUNE>(a, S, chunk, ws, dec.plan, (uint32_t)uniform(in.rnd), (uint32_t)uniform(in.seq), free_words(d, ws, b), round);
}

// ---------------------------------------------------------------------------------------------
// Column-sharded sampling.  Every holder scans its columns under the plan of the (replicated) decision
// stage and exports one record per sequence (best key, its vocabulary index, runner-up key, margin of
// the best); the records of all holders give the winner, or a threshold below which nothing can win;
// the holders then export the few elements above it and the refined normaliser sums of their columns,
// and the float64 keys decide.
// ---------------------------------------------------------------------------------------------
constexpr int kShardCand = 8;          // candidates a holder exports per sequence
struct ShardCand {                     // 128 bytes
  double sum_p, sum_q;                 // sum of 2^(z log2 e - c) over the holder's columns, c = the plan's normalisers
  int32_t n, flags;                    // flags: 1 more candidates than the record holds, 2 the sums are float64-exact
  struct Cand { int32_t idx; float zp, zq; } c[kShardCand];
  int32_t pad[2];
};
static_assert(sizeof(ShardCand) == 128, "exchange record of the sharded refinement");

template <int DT>
__global__ void __launch_bounds__(kBlock, 5) k_shard_scan(SampleArgs a, int S, int col0, Workspace ws) {
  const int b = blockIdx.y, s = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const SamplePlan plan = ws.plan[b];
  if (!plan.valid) return;
  const int V = a.map.V;
  const char* prow = a.map.base[0] + ((int64_t)b * a.map.seq_stride[0] +
                                      (int64_t)plan.row * a.map.pos_stride[0]) * Elem<DT>::bytes;
  const char* qrow = a.map.base[1] + ((int64_t)b * a.map.seq_stride[1] +
                                      (int64_t)plan.row * a.map.pos_stride[1]) * Elem<DT>::bytes;
  const uint32_t c1 = (uint32_t)plan.row | (1u << 16);
  const uint32_t c2 = a.round ? a.round[b] : a.round0;
  const uint32_t c3 = a.seq_id ? a.seq_id[b] : (uint32_t)b;
  const int nv = vectors_of<DT>(V), chunk = slice_chunk(nv, S), v0 = min(s * chunk, nv), v1 = min(v0 + chunk, nv);
  Top2 best{-INFINITY, -1, -INFINITY, -1};
  bool poison = false;
  __shared__ Floors sh_floors;
  scan_plan<DT, false, false>(plan, prow, qrow, V, v0, v1, col0, c1, c2, c3, a.seed_lo, a.seed_hi, best, sh_floors, poison);
  __shared__ Top2 sh_top[kWaves];
  __shared__ int sh_flag[kWaves];
  best = top2_wave_reduce(best);
  const int any_poison = __any(poison);
  if (lane == 0) {
    sh_top[wave] = best;
    sh_flag[wave] = any_poison;
  }
  __syncthreads();
  if (tid == 0) {
    Top2 t = sh_top[0];
    int flag = sh_flag[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) {
      t = top2_merge(t, sh_top[w]);
      flag |= sh_flag[w];
    }
    t.i2 = flag ? -2 : -1;
    ws.part3[(size_t)b * kMaxSampleSplit + s] = t;      // read by the next kernel
  }
}

// One wavefront per sequence: the holder's record (k1, index, k2, margin of its best element).
template <int DT>
__global__ void __launch_bounds__(kBlock) k_shard_fold_top(SampleArgs a, int S, int col0, Workspace ws, float4* out) {
  const int lane = threadIdx.x & 63, b = blockIdx.x * kWaves + (threadIdx.x >> 6);
  if (b >= a.map.B) return;
  const SamplePlan plan = ws.plan[b];
  if (!plan.valid) {
    if (lane == 0) out[b] = make_float4(-INFINITY, __int_as_float(-1), -INFINITY, 0.f);
    return;
  }
  Top2 t{-INFINITY, -1, -INFINITY, -1};
  int flag = 0;
  for (int j = lane; j < S; j += 64) {
    Top2 o = ws.part3[(size_t)b * kMaxSampleSplit + j];
    if (o.i2 == -2) { flag = 1; o.i2 = -1; }
    t = top2_merge(t, o);
  }
  t = top2_wave_reduce(t);
  flag = __any(flag);
  if (lane != 0) return;
  float margin = 0.f;
  if (t.i1 >= 0 && plan.residual == kResidual) {
    const char* prow = a.map.base[0] + ((int64_t)b * a.map.seq_stride[0] +
                                        (int64_t)plan.row * a.map.pos_stride[0]) * Elem<DT>::bytes;
    const char* qrow = a.map.base[1] + ((int64_t)b * a.map.seq_stride[1] +
                                        (int64_t)plan.row * a.map.pos_stride[1]) * Elem<DT>::bytes;
    const float p = ex2(fmaf(load_elem<DT>(prow, t.i1 - col0), kLog2e, -(float)plan.lse2_p));
    const float q = ex2(fmaf(load_elem<DT>(qrow, t.i1 - col0), kLog2e, -(float)plan.lse2_q));
    const float err = kErrRel * (p + q), w = p - q;
    margin = (w > 2.f * err) ? 3.f * kLog2e * err / w : INFINITY;     // INFINITY: the mass of the best is not certain
  }
  out[b] = make_float4(t.k1, __int_as_float(flag ? -2 : t.i1), t.k2, margin);
}

// Replicated.  One wavefront per sequence, one lane per holder: the winner if it is certain, else the
// provisional winner and the threshold tau that a candidate's upper-bound key has to reach.
__global__ void __launch_bounds__(kBlock) k_shard_pick(int B, int G, const float4* top_all, Workspace ws,
                                                       int32_t* next_token, uint32_t* status, float* tau_out) {
  const int lane = threadIdx.x & 63, b = blockIdx.x * kWaves + (threadIdx.x >> 6);
  if (b >= B) return;
  const SamplePlan plan = ws.plan[b];
  float4 rec = make_float4(-INFINITY, __int_as_float(-1), -INFINITY, 0.f);
  if (lane < G) rec = top_all[(size_t)lane * B + b];
  const int idx = __float_as_int(rec.y);
  const int poison = __any(idx == -2);
  Top2 t{rec.x, idx < 0 ? -1 : idx, rec.z, -1};
  if (idx < 0) t.k1 = -INFINITY;
  t = top2_wave_reduce(t);
  const unsigned long long owner = __ballot(t.i1 >= 0 && idx == t.i1);
  const float margin_owner = __shfl(rec.w, owner ? __ffsll((long long)owner) - 1 : 0);
  if (lane != 0) return;
  float tau = INFINITY;                 // nothing to refine
  if (!plan.valid) {
    next_token[b] = -1;                 // the status already says why
  } else if (poison) {
    next_token[b] = -1;
    status[b] |= ADASD_ST_NONFINITE;
  } else if (t.i1 < 0 || !(margin_owner < INFINITY)) {
    next_token[b] = t.i1;               // no element with certain mass: this path cannot settle it
    status[b] |= ADASD_ST_UNSETTLED;
  } else {
    const float margin = kGuard + margin_owner;
    next_token[b] = t.i1;
    if (!(t.k1 - t.k2 > margin)) tau = t.k1 - margin;
  }
  tau_out[b] = tau;
}

// One workgroup per sequence still open (finite tau): the holder's candidates and refined sums.
template <int DT>
__global__ void __launch_bounds__(kBlock) k_shard_refine(SampleArgs a, int S, int col0, const float* tau_in, int exact,
                                                         Workspace ws, ShardCand* out) {
  const int b = blockIdx.x, tid = threadIdx.x;
  const float tau = tau_in[b];
  ShardCand* rec = out + b;
  if (!(tau < INFINITY)) {
    if (tid == 0) {
      rec->sum_p = rec->sum_q = 0.0;
      rec->n = rec->flags = 0;
    }
    return;
  }
  const SamplePlan plan = ws.plan[b];
  const int V = a.map.V;
  const char* prow = a.map.base[0] + ((int64_t)b * a.map.seq_stride[0] +
                                      (int64_t)plan.row * a.map.pos_stride[0]) * Elem<DT>::bytes;
  const char* qrow = a.map.base[1] + ((int64_t)b * a.map.seq_stride[1] +
                                      (int64_t)plan.row * a.map.pos_stride[1]) * Elem<DT>::bytes;
  const uint32_t c1 = (uint32_t)plan.row | (1u << 16);
  const uint32_t c2 = a.round ? a.round[b] : a.round0;
  const uint32_t c3 = a.seq_id ? a.seq_id[b] : (uint32_t)b;
  const bool residual = plan.residual == kResidual;
  __shared__ RefineShared R;
  __shared__ double sh_red[kWaves];
  const bool ok = refine_gather<DT>(prow, qrow, residual, plan.residual == kExclude ? plan.excluded : -1, V, col0, b, S,
                                    tau, (float)plan.lse2_p, (float)plan.lse2_q, c1, c2, c3, a.seed_lo, a.seed_hi, ws, R);
  double sum_p = 0.0, sum_q = 0.0;
  if (residual && exact) {           // every term in float64 (a second attempt after overlapping bounds)
    double ap = 0.0, aq = 0.0;
    for (int v = tid; v < V; v += kBlock) {
      ap += exp((double)load_elem<DT>(prow, v) - plan.lse2_p * 0.69314718055994530942);
      aq += exp((double)load_elem<DT>(qrow, v) - plan.lse2_q * 0.69314718055994530942);
    }
    sum_p = block_sum_d(ap, sh_red);
    sum_q = block_sum_d(aq, sh_red);
  } else if (residual) {
    sum_p = row_pow2_sum_refined<DT>(prow, V, plan.lse2_p, sh_red);
    sum_q = row_pow2_sum_refined<DT>(qrow, V, plan.lse2_q, sh_red);
  }
  const int n = R.n_cand;
  if (tid == 0) {
    rec->sum_p = sum_p;
    rec->sum_q = sum_q;
    rec->n = min(n, kShardCand);
    rec->flags = ((!ok || n > kShardCand) ? 1 : 0) | (exact ? 2 : 0);
  }
  if (tid < min(n, kShardCand)) {
    const int gv = R.cand[tid];
    rec->c[tid].idx = gv;
    rec->c[tid].zp = load_elem<DT>(prow, gv - col0);
    rec->c[tid].zq = residual ? load_elem<DT>(qrow, gv - col0) : 0.f;
  }
}

// Replicated.  One wavefront per sequence: float64 keys of all holders' candidates; the best is final if
// no other can overtake it within the error bounds of the refined normalisers.
__global__ void __launch_bounds__(kBlock) k_shard_settle(SampleArgs a, int G, float* tau_in, const ShardCand* all,
                                                         Workspace ws) {
  const int lane = threadIdx.x & 63, b = blockIdx.x * kWaves + (threadIdx.x >> 6), B = a.map.B;
  if (b >= B) return;
  if (!(tau_in[b] < INFINITY)) return;
  const SamplePlan plan = ws.plan[b];
  const bool residual = plan.residual == kResidual;
  const uint32_t c1 = (uint32_t)plan.row | (1u << 16);
  const uint32_t c2 = a.round ? a.round[b] : a.round0;
  const uint32_t c3 = a.seq_id ? a.seq_id[b] : (uint32_t)b;
  double sp = 0.0, sq = 0.0;
  int overflow = 0, total = 0, exact = 2;
  for (int g = 0; g < G; ++g) {                 // same order on every replica
    const ShardCand* r = all + (size_t)g * B + b;
    sp += r->sum_p;
    sq += r->sum_q;
    overflow |= r->flags & 1;
    exact &= r->flags;
    total += r->n;
  }
  // what the remaining error of the normalisers can do to ln w, per unit of (p + q) / w: one float ulp
  // per term of the refined sums, rounding of float64 sums over the vocabulary for the exact ones
  const double bound = exact ? 0x1p-40 : 0x1p-21;
  const double lse_p = residual ? (plan.lse2_p + log(sp) * 1.44269504088896340736) * 0.69314718055994530942 : 0.0;
  const double lse_q = residual ? (plan.lse2_q + log(sq) * 1.44269504088896340736) * 0.69314718055994530942 : 0.0;
  // candidate number `lane`, `lane + 64`, ... in holder order; float64 key of one of them
  auto key_of = [&](const ShardCand::Cand& e, double* err, uint32_t* word) {
    const int v = e.idx;
    const U4 w4 = philox4x32_10((uint32_t)v >> 2, c1, c2, c3, a.seed_lo, a.seed_hi);
    *word = pick_word(w4, v);
    const double u = ((double)*word + 0.5) * (1.0 / 4294967296.0);
    const double gn = log(-log(u));
    *err = 0.0;
    if (!residual) return (double)e.zp - gn;
    const double p = exp((double)e.zp - lse_p), q = exp((double)e.zq - lse_q);
    const double w = p - q;
    *err = w > 0.0 ? bound * (p + q) / w : INFINITY;
    return w > 0.0 ? log(w) - gn : -INFINITY;
  };
  // pass 1: the best key (lowest index among equal ones), with the inputs it was formed from
  double best_key = -INFINITY, best_err = 0.0;
  int best_idx = 0x7fffffff, uncertain = 0;
  float best_zp = 0.f, best_zq = 0.f;
  uint32_t best_word = 0u;
  int seen = 0;
  for (int g = 0; g < G; ++g) {
    const ShardCand* r = all + (size_t)g * B + b;
    for (int c = 0; c < r->n; ++c, ++seen) {
      if ((seen & 63) != lane) continue;
      double err;
      uint32_t word;
      const double key = key_of(r->c[c], &err, &word);
      if (residual && !(err < 0.25)) uncertain = 1;
      const int v = r->c[c].idx;
      if (key > best_key || (key == best_key && v < best_idx)) {
        best_key = key;
        best_err = err;
        best_idx = v;
        best_zp = r->c[c].zp;
        best_zq = r->c[c].zq;
        best_word = word;
      }
    }
  }
  double wk = best_key;
  int wi = best_idx;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const double ok = __shfl_xor(wk, off);
    const int oi = __shfl_xor(wi, off);
    if (ok > wk || (ok == wk && oi < wi)) { wk = ok; wi = oi; }
  }
  const unsigned long long owner_mask = __ballot(best_idx == wi && best_key == wk);
  const int owner = owner_mask ? __ffsll((long long)owner_mask) - 1 : 0;
  const double werr = __shfl(best_err, owner);
  const float wzp = __shfl(best_zp, owner), wzq = __shfl(best_zq, owner);
  const uint32_t wword = (uint32_t)__shfl((int)best_word, owner);
  // pass 2: the largest upper end among the others.  A candidate formed from the very same logits and the
  // very same noise word as the winner has the winner's key whatever the normalisers are: an exact tie,
  // which the lower index wins, not a close call.
  double others = -INFINITY;
  seen = 0;
  for (int g = 0; g < G; ++g) {
    const ShardCand* r = all + (size_t)g * B + b;
    for (int c = 0; c < r->n; ++c, ++seen) {
      if ((seen & 63) != lane || r->c[c].idx == wi) continue;
      double err;
      uint32_t word;
      const double key = key_of(r->c[c], &err, &word);
      if (word == wword && r->c[c].zp == wzp && r->c[c].zq == wzq) continue;
      others = fmax(others, key + err);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) others = fmax(others, __shfl_xor(others, off));
  uncertain = __any(uncertain);
  if (lane != 0) return;
  if (total == 0 || overflow || uncertain || wi == 0x7fffffff || (residual && !(wk - werr > others))) {
    // the provisional token of the pick stage stays; tau stays finite, so another refine + settle
    // with exact sums can still close it
    a.status[b] |= ADASD_ST_UNSETTLED;
  } else {
    a.next_token[b] = wi;
    a.status[b] = (a.status[b] & ~(uint32_t)ADASD_ST_UNSETTLED) | ADASD_ST_EXACT_PATH;
    tau_in[b] = INFINITY;
  }
}

}  // namespace

hipError_t launch_sample(const SampleArgs& a, int S, const Workspace& ws, hipStream_t st) {
  if (a.map.B <= 0) return hipSuccess;
  const dim3 grid(S, a.map.B), block(kBlock);
  const int epv = a.dt == ADASD_BF16 ? 8 : 4, chunk = slice_chunk((a.map.V + epv - 1) / epv, S);
  const bool slices = S > kMaxSplit, prune = scan_prunes(chunk, a.dt);
#define ADASD_SAMPLE_CASE(DTV, LONGV, PRUNEV) \
  if (a.dt == DTV && slices == LONGV && prune == PRUNEV) launch_kernel((k_sample<DTV, LONGV, PRUNEV>), grid, block, st, a, S, chunk, ws);
  ADASD_SAMPLE_CASE(ADASD_BF16, false, false) ADASD_SAMPLE_CASE(ADASD_BF16, false, true)
  ADASD_SAMPLE_CASE(ADASD_BF16, true, false) ADASD_SAMPLE_CASE(ADASD_BF16, true, true)
  ADASD_SAMPLE_CASE(ADASD_F32, false, false) ADASD_SAMPLE_CASE(ADASD_F32, false, true)
  ADASD_SAMPLE_CASE(ADASD_F32, true, false) ADASD_SAMPLE_CASE(ADASD_F32, true, true)
#undef ADASD_SAMPLE_CASE
  return hipGetLastError();
}

// Deciding in every workgroup of the token scan takes about as long as deciding in one while each workgroup has a
// compute unit (or, without appends inside the loop, half of one) to itself; then it saves a launch.  Beyond that the workgroups
// hold one another up.  Windows above 8 would take a second turn of the positions; long histories have their own kernel;
// the slices' words need room beside those of the statistics kernel.  Whole calls (us), two kernels / one: 1 x 4 x 32000
// float 17.3 / 16.2, 1 x 8 x 128256 19.8 / 18.9, 4 x 4 x 128256 20.4 / 19.0, 16 x 6 x 32003 literal 22.4 / 20.7; 504
// workgroups (8 x 8 x 128256) 27.4 / 26.5, 512 (16 x 8 x 32000) 23.8 / 22.4, literal 512 (32 x 4 x 32003) 22.5 / 23.0;
// 1008 (16 x 8 x 128256) 37.8 / 38.6, 2016 55.0 / 56.1.
bool merges_decisions(const DecideArgs& d, int S) {
  const int free_slots = kMaxSplit - d.xchg_split;
  const bool wide = d.cap >= kWideCap && !d.relaxed_off && d.LA && d.LR && d.nA && d.nR;
  const bool hist = d.hist != nullptr || d.relaxed_off || !(d.LA && d.LR && d.nA && d.nR);
  return d.xchg_split > 0 && hist && !wide && d.map.K <= 8 && S <= kMaxSplit && 2 * free_slots >= kMaxSplit &&
         S <= (d.map.K > 1 ? kMaxSplit : free_slots) && S * d.map.B <= (d.list_update ? kMergeInLoop : kMergeGroups);
}

hipError_t launch_decide_sample(const DecideArgs& d, const UpdateArgs& upd, const SampleArgs& a, int S, const Workspace& ws, hipStream_t st) {
  if (a.map.B <= 0) return hipSuccess;
  const dim3 grid(S, a.map.B), block(kBlock);
  const int epv = a.dt == ADASD_BF16 ? 8 : 4, chunk = slice_chunk((a.map.V + epv - 1) / epv, S);
  const bool prune = scan_prunes(chunk, a.dt);
  const int LP = d.map.K <= 4 ? 64 : 32;
#define ADASD_MERGED_CASE(DTV, INLOOPV, LPV, PRUNEV) \
  if (a.dt == DTV && (d.list_update != 0) == INLOOPV && LP == LPV && prune == PRUNEV) \
    launch_kernel((k_decide_sample<DTV, INLOOPV, LPV, PRUNEV>), grid, block, st, d, upd, a, S, chunk, ws);
#define ADASD_MERGED_DT(DTV) \
  ADASD_MERGED_CASE(DTV, false, 32, false) ADASD_MERGED_CASE(DTV, false, 32, true) \
  ADASD_MERGED_CASE(DTV, true, 32, false) ADASD_MERGED_CASE(DTV, true, 32, true) \
  ADASD_MERGED_CASE(DTV, false, 64, false) ADASD_MERGED_CASE(DTV, false, 64, true) \
  ADASD_MERGED_CASE(DTV, true, 64, false) ADASD_MERGED_CASE(DTV, true, 64, true)
  ADASD_MERGED_DT(ADASD_BF16)
  ADASD_MERGED_DT(ADASD_F32)
#undef ADASD_MERGED_DT
#undef ADASD_MERGED_CASE
  return hipGetLastError();
}

hipError_t launch_shard_sample(const SampleArgs& a, int S, int col0, const Workspace& ws, float4* top_out, hipStream_t st) {
  if (a.map.B <= 0) return hipSuccess;
  const dim3 grid(S, a.map.B), block(kBlock), fold((a.map.B + kWaves - 1) / kWaves);
  if (a.dt == ADASD_BF16) {
    launch_kernel(k_shard_scan<ADASD_BF16>, grid, block, st, a, S, col0, ws);
    launch_kernel(k_shard_fold_top<ADASD_BF16>, fold, block, st, a, S, col0, ws, top_out);
  } else {
    launch_kernel(k_shard_scan<ADASD_F32>, grid, block, st, a, S, col0, ws);
    launch_kernel(k_shard_fold_top<ADASD_F32>, fold, block, st, a, S, col0, ws, top_out);
  }
  return hipGetLastError();
}

hipError_t launch_shard_pick(int B, int G, const float4* top_all, const Workspace& ws, int32_t* next_token,
                             uint32_t* status, float* tau_out, hipStream_t st) {
  if (B <= 0) return hipSuccess;
  launch_kernel(k_shard_pick, dim3((B + kWaves - 1) / kWaves), dim3(kBlock), st, B, G, top_all, ws, next_token, status, tau_out);
  return hipGetLastError();
}

hipError_t launch_shard_refine(const SampleArgs& a, int S, int col0, const float* tau, int exact, const Workspace& ws,
                               void* cand_out, hipStream_t st) {
  if (a.map.B <= 0) return hipSuccess;
  if (a.dt == ADASD_BF16)
    launch_kernel(k_shard_refine<ADASD_BF16>, dim3(a.map.B), dim3(kBlock), st, a, S, col0, tau, exact, ws, static_cast<ShardCand*>(cand_out));
  else
    launch_kernel(k_shard_refine<ADASD_F32>, dim3(a.map.B), dim3(kBlock), st, a, S, col0, tau, exact, ws, static_cast<ShardCand*>(cand_out));
  return hipGetLastError();
}

hipError_t launch_shard_settle(const SampleArgs& a, int G, float* tau, const void* cand_all, const Workspace& ws,
                               hipStream_t st) {
  if (a.map.B <= 0) return hipSuccess;
  launch_kernel(k_shard_settle, dim3((a.map.B + kWaves - 1) / kWaves), dim3(kBlock), st, a, G, tau,
                static_cast<const ShardCand*>(cand_all), ws);
  return hipGetLastError();
}

}  // namespace adasd
