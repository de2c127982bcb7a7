// The drafting calls of the generation loop of Algorithm 1, each ONE launch and one pass over the
// logits: entropy of the draft row (Appendix A), stop rule H(q_i) > T_G (Section 4.3) and, for
// adasd_draft_step, the token x_i ~ q_i.  The Gumbel-max key of an element, ln q_v - ln(-ln u_v),
// differs from z_v - ln(-ln u_v) only by the row's normaliser, so the argmax needs no second pass: the
// scan forms the entropy sums and the keys from the same registers.  One workgroup of a row folds
// the row's slice records and settles close calls of the argmax in float64.
#include "sample_device.h"
#include "stats_device.h"

namespace adasd {

namespace {

using namespace sampling;

// One wavefront folds its lanes' states: common reference (which carries the valid flag of the hand-off words),
// plain sums, winner and runner-up.  Uniform results.
template <bool DRAW> __device__ __forceinline__ void fold_wave(Lse& l, Top2& t) {
  float top = l.m, best = t.k1;
  if (DRAW) wave_max2(top, best);              // (one chain of exchanges for both)
  else top = wave_max_f(top);
  const float M = __uint_as_float(__float_as_uint(top) | 1u);
  const float d = top > kNegHuge ? l.m - M : 0.f, f = ex2(d);     // (nothing finite seen: the sums are 0, or a NaN)
  float a = l.s * f, b = (l.u + d * l.s) * f;
  swap32(a, b);
  float x = a + b, y = x;
  swap16(x, y);
  x = row_sum16(x + y);                        // lower half of the lanes: the sum, upper half: the weighted sum
  l = Lse{M, lane_value(x, 0), lane_value(x, 32)};
  if (DRAW) t = top2_below(t, best);
}
// The same of the workgroup's wavefronts, whose states (folded, with references that carry the flag) are in shared memory: every
// lane goes through them by itself, which is shorter than the exchanges between lanes (0.18 us of a drafting call of 1 x 32000 float).
template <bool DRAW> __device__ __forceinline__ void fold_workgroup(const Lse (&ls)[kWaves], const Top2 (&ts)[kWaves], Lse& l, Top2& t) {
  float M = ls[0].m;
#pragma unroll
  for (int w = 1; w < kWaves; ++w) M = fmaxf(M, ls[w].m);
  float s[kWaves], u[kWaves];
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const float d = M > kNegHuge ? ls[w].m - M : 0.f, f = ex2(d);
    s[w] = ls[w].s * f;
    u[w] = (ls[w].u + d * ls[w].s) * f;
  }
  l = Lse{__uint_as_float(__float_as_uint(M) | 1u), (s[0] + s[1]) + (s[2] + s[3]), (u[0] + u[1]) + (u[2] + u[3])};
  if (DRAW) t = top2_merge(top2_merge(ts[0], ts[1]), top2_merge(ts[2], ts[3]));
}

// Sums of a whole row by one wavefront, from the logits (where the slices' records did not arrive, which never happens
// to calls that are ordered as they have to be).
template <int DT> __device__ __forceinline__ Lse wave_row_sums(const char* row, int V) {
  const int lane = threadIdx.x & 63;
  float top = kNegHuge;
#pragma unroll 1
  for (int v = lane; v < V; v += 64) {
    const float z = load_elem<DT>(row, v);
    if (z < INFINITY) top = fmaxf(top, z);
  }
  top = wave_max_f(top);
  const float m = top > kNegHuge ? top * kLog2e : kNegHuge;
  double s = 0.0, u = 0.0;
#pragma unroll 1
  for (int v = lane; v < V; v += 64) {
    const float t = fmaf(load_elem<DT>(row, v), kLog2e, -m), e = ex2(t);
    s += (double)e;
    u += (double)fmaxf(t, -200.f) * (double)e;            // (masked logits: 0; a broken one shows in s)
  }
  return Lse{m, (float)wave_sum(s), (float)wave_sum(u)};
}

struct DraftShared {
  Floors floors;
  Lse l[kWaves];
  Top2 t[kWaves];
  int mode;      // 0 another workgroup folds the row; 1 final; 2 settle among the close candidates;
                 // 3 broken row; 4 whole row in float64; 5 the same, and the entropy from the logits too
  float tau;
  double red[kWaves];
};

// What a drafting call has to do per logit is: 3 plain instructions and an exponential for the entropy, 18
// multiplications and 19 exclusive ors per four logits for the noise, and for the key two conversions, two logarithms
// and about a dozen more; from four groups of logits per wavefront on, the key's part is only done where the logit may
// still win (PRUNE: three instructions to find out; the kernel alone, 128 rows of 152064 25.8 -> 21.5 us, 896 of 128256
// 108 -> 77).  While the wavefronts run it is bound by the vector ALU, so everything here follows the issue
// rules of device_common.h; the slices are cut so that the whole call is resident at once with equal shares per thread.  A wavefront
// of 128 rows of 152064 lives 12.3 of the call's 20.3 us, 44 % of it waiting for its turn to issue and 29 % for memory; one of 24
// rows of 128256 about 6 of 8.2, 23 % and 47 %.  The rest of a call is its start, its hand-off and that not all end at once.
// Back to back, bf16, against loops that alternated transcendentals with plain instructions and took the slices in
// batches of vectors: 128 rows of 152064 39.0 -> 24.3 us, 24 of 32 rows of 128256 11.1 -> 8.9 us; one row of 128256
// 8.8 -> 6.0 us (3.4 us of it are the host's part of the call, which runs beside the kernel of the call before).
// With few rows it is a chain of latencies: 0.6 us to the first logits, 0.6 to 0.9 for the scan, 0.5 for the wavefronts' and the
// workgroup's fold, 0.6 until the last slice's record has arrived, 0.5 for the row's fold and the results.  The wavefronts
// without logits behind a row's end stood in it with 1 us (top2_below), the ticket with 0.4, the threshold, asked for
// when it was needed, with 0.3: 1 x 128256 bf16 5.95 -> 4.65 us a call, 1 x 32000 float 5.96 -> 4.35, 24 of 32 rows of 128256 8.82 ->
// 8.20, entropies of 32 x 128256 float 6.57 -> 6.17.  (More than one vector ahead on its way: 6.2 -> 6.4 us with the entropies, 8.4 -> 8.5 with the draw.)
//
// One launch per drafting call, grid (slices, rows).  One workgroup of a row (few_rows) folds
// the slices' records, and with DRAW settles a winner that does not lead by more than the rounding guard.
template <int DT, bool DRAW, bool PRUNE>
__global__ void __launch_bounds__(kBlock, 7) k_draft(RowMap map, int S, int chunk, Workspace ws, DraftOut dout, DraftDraw dr) {
  warm_kernargs<sizeof(RowMap) + 2 * sizeof(int) + sizeof(Workspace) + sizeof(DraftOut) + sizeof(DraftDraw)>();
  constexpr int EPV = Elem<DT>::per_vec;
  __shared__ DraftShared sh;
  const int rho = blockIdx.y, s = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const RowRef r = locate_row<DT>(map, rho);

  // ---- the slice: vectors v0 .. v1 of the row, one per thread and turn, the next one always on its way
  const int V = map.V, nv = vectors_of<DT>(V), whole = V / EPV;
  const int v0 = min(s * chunk, nv), v1 = min(v0 + chunk, nv);
  const uint4 neutral = neutral_vec<DT>();
  auto load = [&](int idx) {
    uint4 x = neutral;
    if (idx < v1) {
      if (idx < whole) x = load_vec_any(r.ptr, idx);
      else x = load_last_vec<DT>(r.ptr, V);
    }
    return x;
  };
  if (!r.active) {
    if (s == 0 && tid == 0) {
      dout.H_out[rho] = 0.f;
      if (dout.stop_out) dout.stop_out[rho] = 0;
      if (DRAW) {
        dr.token_out[rho] = -1;
        if (dr.status) dr.status[rho] = 0;
      }
    }
    return;
  }
  // (only here: the logits of a row at rest need not be there)
  uint4 next = load(v0 + tid);
  // (needed at the very end, where it was a latency of its own; ahead of the row it would be one too)
  const float threshold = dout.T_G ? scalar_load(dout.T_G + rho) : INFINITY;
  const uint32_t c1 = dr.step | (2u << 16);
  const uint32_t c2 = DRAW ? (dr.round ? scalar_load(dr.round + rho) : dr.round0) : 0u;
  const uint32_t c3 = DRAW ? (dr.seq_id ? scalar_load(dr.seq_id + rho) : (uint32_t)rho) : 0u;
  if (PRUNE) floors_init(sh.floors);
  PhiloxRow noise;
  if (DRAW) noise = philox_row(c1, c2, c3, dr.seed_lo, dr.seed_hi);
  Lse st = lse_empty();
  Top2 best{-INFINITY, -1, -INFINITY, -1};
  float floor = kNoFloor;        // (uniform in the wavefront) see may_win
  for (int base = v0; base < v1; base += kBlock) {
    const uint4 x = next;
    const int idx = base + tid;
    if (base + kBlock < v1) next = load(idx + kBlock);
    // the lane's own reference follows its largest logit; the vector's sums are formed on their own and then join the
    // lane's (a chain of additions over all of a lane's logits would round once more per logit: a row of 32000 in one
    // slice had its entropy to 6.1e-8 rms that way, 4.4e-8 this way)
    const uint4 one[1] = {x};
    const float m = fmaxf(st.m, vecs_max<DT, 1>(one)), d = st.m - m, f = ex2(d), neg_m = -m;
    st.u = (st.u + d * st.s) * f;
    st.s *= f;
    st.m = m;
    if (base + (tid & ~63) >= v1) continue;     // (a whole wavefront past the end)
    if (PRUNE) floor = highest_floor(sh.floors, floor);
    float s0 = 0.f, s1 = 0.f, u0 = 0.f, u1 = 0.f;
#pragma unroll
    for (int g = 0; g < EPV / 4; ++g) {
      float z[4], t[4], e[4];
      unpack4<DT>(x, g, z);
#pragma unroll
      for (int i = 0; i < 4; ++i) t[i] = fma_log2e(z[i], neg_m);
      ex2_group(t, e);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float &s = i & 1 ? s1 : s0, &u = i & 1 ? u1 : u0;
        s = g == 0 && i < 2 ? e[i] : s + e[i];
        // masked logits: (-200) * 0 = 0; a NaN stays one through e
        u = g == 0 && i < 2 ? max_raw(t[i], -200.f) * e[i] : fmaf(max_raw(t[i], -200.f), e[i], u);
      }
      if (DRAW) {
        const int first = idx * EPV + 4 * g;
        const U4 block = philox_block(noise, (uint32_t)first >> 2);
        if (!PRUNE || may_win(e, reach(m, floor), block)) {
          float lE[4];
          log2_exponential4(block, lE);
#pragma unroll
          for (int i = 0; i < 4; ++i) top2_push(best, fma_log2e(z[i], -lE[i]), first + i);   // (a masked logit: -inf, never the best)
          if (PRUNE) floor = raise_floor(sh.floors, floor, best.k1);
        }
      }
    }
    st.s += s0 + s1;
    st.u += u0 + u1;
  }

  auto write_row = [&](const RowResult& res) {
    dout.H_out[rho] = res.H;
    if (dout.stop_out) {
      dout.stop_out[rho] = (uint8_t)(res.H > threshold || dout.force_stop || res.bad);
    }
  };

  // ---- the slice's record
  fold_wave<DRAW>(st, best);
  if (lane == 0) {
    sh.l[wave] = st;
    if (DRAW) sh.t[wave] = best;
  }
  __syncthreads();
  if (wave == 0) {
    fold_workgroup<DRAW>(sh.l, sh.t, st, best);
    bool last = true, arrived = true;
    uint64_t w[kXchgWords];
    if (S > 1) {
      pack_draft(DraftRecord{st.m, st.s, st.u, best.k1, best.k2, best.i1}, w);
      last = hand_off(PlainWords{ws.xchg + (size_t)rho * kMaxSplit * kXchgWords}, s, S, Arrivals{ws.ticket1, kTicket1Len, rho, map.B},
                      dout.wait, [] {}, w, arrived);
    }
    if (last) {
      // ---- the row's records folded
      if (S > 1) {
        st = lse_empty();
        best = Top2{-INFINITY, -1, -INFINITY, -1};
        if (lane < S) {
          const DraftRecord rec = unpack_draft(w);
          st = Lse{rec.m, rec.s, rec.u};
          best = Top2{rec.k1, rec.i1, rec.k2, -1};
        }
      } else if (lane != 0) {
        st = lse_empty();
        best = Top2{-INFINITY, -1, -INFINITY, -1};
      }
      const Top2 mine = best;
      fold_wave<DRAW>(st, best);
      const RowResult res = finish_row(st);
      int mode = 1;
      if (DRAW) {
        if (!arrived) mode = 5;
        else if (res.bad) mode = 3;
        else if (best.i1 < 0) mode = 4;
        else if (!(best.k1 - best.k2 > kGuard)) mode = 2;
        if (mode == 2 && lane < S) {          // the slices' records, for the search for close candidates
          Top2* dst = &ws.part3[(size_t)rho * kMaxSampleSplit + lane];
          st_agent(&dst->k1, mine.k1);
          st_agent(&dst->i1, mine.i1);
          st_agent(&dst->k2, mine.k2);
          publish_barrier();
        }
      }
      if (lane == 0) {
        write_row(res);
        if (DRAW && (mode == 1 || mode == 3)) {
          dr.token_out[rho] = mode == 1 ? best.i1 : -1;
          if (dr.status) dr.status[rho] = mode == 1 ? 0u : (uint32_t)ADASD_ST_NONFINITE;
        }
        sh.mode = mode;
        sh.tau = best.k1 - kGuard;
      }
      if (!DRAW && __builtin_expect(!arrived, 0)) {
        const RowResult whole = finish_row(wave_row_sums<DT>(r.ptr, V));
        if (lane == 0) write_row(whole);
      }
    } else if (lane == 0) {
      sh.mode = 0;
    }
  }
  if (!DRAW) return;
  __syncthreads();
  const int mode = sh.mode;
  if (mode == 0 || mode == 1 || mode == 3) return;
  if (mode == 5 && wave == 0) {
    const RowResult whole = finish_row(wave_row_sums<DT>(r.ptr, V));
    if (lane == 0) write_row(whole);
  }
  uint32_t bits = ADASD_ST_EXACT_PATH;
  int tok = -1;
  if (mode == 2) {
    __shared__ RefineShared sh_refine;
    tok = sample_refine<DT>(r.ptr, nullptr, kPlain, -1, V, rho, S, sh.tau, 0.f, 0.f, 0.0, 0.0, c1, c2, c3,
                            dr.seed_lo, dr.seed_hi, ws, sh.red, sh_refine);
  }
  if (tok < 0)
    tok = sample_exact<DT>(r.ptr, nullptr, false, -1, V, c1, c2, c3, dr.seed_lo, dr.seed_hi, sh.red, &bits);
  if (tid == 0) {
    dr.token_out[rho] = tok;
    if (dr.status) dr.status[rho] = bits;
  }
}

}  // namespace

hipError_t launch_draft_step(const RowMap& map, int dt, const Workspace& ws, const DraftOut& dout,
                             const DraftDraw* draw, hipStream_t st) {
  if (map.B <= 0) return hipSuccess;
  const int S = scan_split(map.B, map.V, dt), epv = dt == ADASD_BF16 ? 8 : 4;
  const int chunk = sampling::slice_chunk((map.V + epv - 1) / epv, S);
  const dim3 grid(S, map.B), block(kBlock);
  const DraftDraw dr = draw ? *draw : DraftDraw{};
  const bool prune = scan_prunes(chunk, dt);
#define ADASD_DRAFT_CASE(DTV, DRAWV, PRUNEV) \
  if (dt == DTV && (draw != nullptr) == DRAWV && (DRAWV && prune) == PRUNEV) \
    launch_kernel((k_draft<DTV, DRAWV, PRUNEV>), grid, block, st, map, S, chunk, ws, dout, dr);
  ADASD_DRAFT_CASE(ADASD_BF16, false, false) ADASD_DRAFT_CASE(ADASD_BF16, true, false) ADASD_DRAFT_CASE(ADASD_BF16, true, true)
  ADASD_DRAFT_CASE(ADASD_F32, false, false) ADASD_DRAFT_CASE(ADASD_F32, true, false) ADASD_DRAFT_CASE(ADASD_F32, true, true)
#undef ADASD_DRAFT_CASE
  return hipGetLastError();
}

}  // namespace adasd
