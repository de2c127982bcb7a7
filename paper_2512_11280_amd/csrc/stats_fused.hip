// Single-read statistics kernel: normalisers, entropies and JS distance of every (target, draft) row
// pair with ONE read of the logits (Appendix A and Section 2.2 of the paper).
//
// The JS distance needs both normalisers before its first term can be formed, so the computation is
// inherently two-phase.  Instead of streaming the rows twice, every thread keeps its few 16-byte
// vectors of the row pair in registers across the two phases.  A work item is one slice of one
// position (T threads x NB vectors per row); a workgroup runs phase 1 on it (reference, sum, weighted
// sum of both rows), publishes the slice's result, waits for the other slices of the position, folds
// all of them (every workgroup of a position the same way, so the same normalisers everywhere) and
// runs phase 2 (the JS sum) on the registers it still holds.
//
// One workgroup per item, T threads, NB vectors per thread and row held in registers from the load to
// the end of phase 2.  What bounds it is the vector ALU: per logit pair 8 plain instructions and two
// exponentials in phase 1, 19 and three transcendentals in phase 2.  The loops over the registers are
// written for the way the SIMDs issue (device_common.h: transcendentals in groups at raised priority,
// per-row constants in vector registers); there are many pairs per thread, because the reductions and the
// exchange cost a fixed number of instructions per item, and with four vectors per thread and row the
// kernel fits 64 registers, i.e. eight wavefronts per SIMD.  Measured (logit pairs of B x k x V, bf16):
// 32 x 8 x 128256 46.6 -> 41 us, 128 x 16 x 152064 388 -> 335 us with the loops written this way.
//
// Hand-off between the workgroups of a position: self-validating 64-bit words (records.h; a cleared word
// is 0) written and read with agent-scope atomic accesses: no fence, no separate flag, no
// read-modify-write, and since every word carries its own validity no ordering between different words is
// relied on.  The decision kernel, which runs next, clears the words of the positions it handles.  The
// slices of a position are consecutive workgroups of the grid and workgroups are dispatched in order, so
// whenever one waits, the ones it waits for are resident or next in line; all the same every wait is
// bounded: after `wait_polls` polls the workgroup recomputes the other slices' results itself from memory
// with the very same code (bit-identical), so every wave exits whatever the dispatch order is.
#include "history_device.h"
#include "stats_device.h"
#include "records.h"

namespace adasd {

namespace {

__device__ __forceinline__ uint64_t get_word(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct FusedGeom {
  int S;           // slices (work items) per position
  int nv;          // 16-byte vectors per row, the last one maybe not whole
  int missing;     // logits that the last vector lacks of a whole one
  int last_byte;   // offset of the last 16 bytes of a row
  int chunk;       // vectors per slice
  int hist_rows;   // rows of the grid, the first ones, that are for the history lists
  int naps;        // naps before the first poll (see kManyGroups)
  int wait_polls;  // polls before a workgroup stops waiting and recomputes what is missing
};

struct SliceRecord {   // phase-1 result of one wavefront or slice: references (they carry the valid flag); S, U of the
  float m[2], v[4];    // target row, S, U of the draft row
};

template <int W> struct FusedShared {
  SliceRecord wave[W];            // per-wavefront results of the slice in hand
  SliceRecord redo[kMaxSplit];    // recomputed slices (only after an expired wait)
  JsNorm norm;
  RowResult row[2];
  int bad, expired;
  float acc[W];
};

// Workgroup barrier that waits for LDS traffic only (outstanding global loads stay in flight).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The vectors of slice s that this thread holds: vector j is number v0 + tid + j*T of the row; a lane past the
// end re-reads the slice's last vector (pad_slice then takes its weight away).  A row may start at any logit and
// have any length: where its last vector is not whole, the row's last 16 bytes are read in its place, and pad_slice
// takes the weight off the logits that the vector before has too.  (Which logit sits where in a vector is of no
// consequence here.)
template <int DT, int T, int NB>
__device__ __forceinline__ void load_slice(const char* prow, const char* qrow, int s, const FusedGeom& g,
                                           uint4 (&xp)[NB], uint4 (&xq)[NB]) {
  const int v0 = min(s * g.chunk, g.nv), v1 = min(v0 + g.chunk, g.nv), tid = threadIdx.x;
  const int last = min(v1 * 16 - 16, g.last_byte);     // (an empty slice reads the row's end for all its lanes)
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int at = min((v0 + tid + j * T) * 16, last);
    xp[j] = load_vec_at(prow, at);
    xq[j] = load_vec_at(qrow, at);
  }
}
// What stands in a lane past the end, once the references are known: a finite logit (-2.3e38) whose exponential
// is 0 against any reference a row can have, so that it adds nothing to any sum and needs no branch.  (An
// infinite one would do the same in the sums of 2^t, but t 2^t has no value there.)
// SKIP: a wavefront leaves out the vectors of which all its lanes are past the end (`left`: vectors of the slice from its first lane
// on).  For slices that leave a wavefront such a vector: whole calls (us) without / with, 64 x 16 x 16392 (half of a workgroup's
// vectors) 48.2 / 39.6, 64 x 16 x 20000 48.6 / 41.7, 32 x 8 x 50257 float 39.2 / 38.5, 64 x 16 x 100000 142 / 134,
// 128 x 16 x 152064 (6 % of them) 369 / 360.  Where there is none the branches cost 32 x 8 x 128256 56.1 -> 56.5.
template <int DT> __device__ __forceinline__ uint32_t weightless() { return DT == ADASD_BF16 ? 0xFF2DFF2Du : 0xFF2D0000u; }
template <int DT, int T, int NB>
__device__ __forceinline__ void pad_slice(int s, const FusedGeom& g, uint4 (&xp)[NB], uint4 (&xq)[NB]) {
  const int v0 = min(s * g.chunk, g.nv), len = min(v0 + g.chunk, g.nv) - v0, tid = threadIdx.x;
  const uint32_t w = weightless<DT>();
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    if ((j + 1) * T <= len) continue;  // (uniform) every lane has its vector
    const bool in = tid + j * T < len;
    xp[j] = make_uint4(in ? xp[j].x : w, in ? xp[j].y : w, in ? xp[j].z : w, in ? xp[j].w : w);
    xq[j] = make_uint4(in ? xq[j].x : w, in ? xq[j].y : w, in ? xq[j].z : w, in ? xq[j].w : w);
  }
  if (g.missing == 0 || v0 + len != g.nv || len == 0) return;     // (uniform)
  // the row's last vector: its first logits are the vector's before
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    if ((len - 1) / T != j) continue;  // (uniform)
    const bool here = tid + j * T == len - 1;
    auto take = [&](int i) -> uint32_t {              // mask of what word i keeps
      if (DT == ADASD_F32) return i < g.missing ? 0u : ~0u;
      return (2 * i < g.missing ? 0u : 0xffffu) | (2 * i + 1 < g.missing ? 0u : 0xffff0000u);
    };
    auto keep = [&](uint32_t x, uint32_t m) { return here ? (x & m) | (w & ~m) : x; };
    const uint32_t m0 = take(0), m1 = take(1), m2 = take(2), m3 = take(3);
    xp[j] = make_uint4(keep(xp[j].x, m0), keep(xp[j].y, m1), keep(xp[j].z, m2), keep(xp[j].w, m3));
    xq[j] = make_uint4(keep(xq[j].x, m0), keep(xq[j].y, m1), keep(xq[j].z, m2), keep(xq[j].w, m3));
  }
}

// Vectors of slice s from the wavefront's first lane on.
__device__ __forceinline__ int wave_left(int s, const FusedGeom& g) {
  const int v0 = min(s * g.chunk, g.nv);
  return min(g.chunk, g.nv - v0) - (__builtin_amdgcn_readfirstlane((int)threadIdx.x) & ~63);
}

__device__ __forceinline__ void record_rows(const SliceRecord& o, Lse& tp, Lse& tq) {
  tp = Lse{o.m[0], o.v[0], o.v[1]};
  tq = Lse{o.m[1], o.v[2], o.v[3]};
}
// Partial states of the two rows, one of each per lane, folded by one wavefront: common reference, plain sums.
// The target row's result in the lower half of the lanes, the draft row's in the upper half.
__device__ __forceinline__ Lse fold_pair(const Lse& tp, const Lse& tq) {
  float mp = tp.m, mq = tq.m;
  wave_max2(mp, mq);
  const float dp = tp.m - mp, dq = tq.m - mq, ep = ex2(dp), eq = ex2(dq);
  float s = wave_sum4(tp.s * ep, tq.s * eq, (tp.u + dp * tp.s) * ep, (tq.u + dq * tq.s) * eq), u = s;
  swap16(s, u);
  return Lse{(threadIdx.x & 32) ? mq : mp, s, u};
}
// The two rows' states from the halves, in every lane.
__device__ __forceinline__ void split_halves(const Lse& f, Lse& tp, Lse& tq) {
  tp = tq = f;
  swap32(tp.m, tq.m);
  swap32(tp.s, tq.s);
  swap32(tp.u, tq.u);
}

// S and U of the wavefront's logits about their references.  MASKED: a logit of -inf is kept from making
// (-inf) * 0 out of its weighted term; without it such a logit turns the weighted sum into a NaN (as a NaN
// does), which the caller sees.
template <int DT, int T, int NB, bool MASKED, bool SKIP>
__device__ __forceinline__ float phase1_sums(const uint4 (&xp)[NB], const uint4 (&xq)[NB], float neg_mp, float neg_mq, int left) {
  float s[2][2] = {{0.f, 0.f}, {0.f, 0.f}}, u[2][2] = {{0.f, 0.f}, {0.f, 0.f}};
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    if (SKIP && j > 0 && j * T >= left) break;
#pragma unroll
    for (int half = 0; half < Elem<DT>::per_vec / 4; ++half)
#pragma unroll
      for (int row = 0; row < 2; ++row) {
        float t[4], e[4];
        unpack4<DT, MASKED>(row ? xq[j] : xp[j], half, t);
#pragma unroll
        for (int i = 0; i < 4; ++i) t[i] = fma_log2e(t[i], row ? neg_mq : neg_mp);
        ex2_group(t, e);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          s[row][i & 1] += e[i];
          u[row][i & 1] = fmaf(MASKED ? fmaxf(t[i], -200.f) : t[i], e[i], u[row][i & 1]);
        }
      }
  }
  return wave_sum4(s[0][0] + s[0][1], s[1][0] + s[1][1], u[0][0] + u[0][1], u[1][0] + u[1][1]);
}

// Phase 1 of the slice held in (xp, xq) by the whole workgroup.  In wavefront 0 the lower half of the lanes
// returns the target row's (m, s, u), the upper half the draft row's; the other wavefronts return nothing of
// use.  One workgroup barrier.  masked: whether a logit of -inf (or a NaN) was met by this wavefront.
template <int DT, int T, int NB, bool SKIP>
__device__ __forceinline__ Lse phase1(int s, const FusedGeom& g, uint4 (&xp)[NB], uint4 (&xq)[NB], bool& masked,
                                      FusedShared<T / 64>& sh) {
  constexpr int W = T / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float mp = vecs_max<DT, NB>(xp), mq = vecs_max<DT, NB>(xq);
  wave_max2(mp, mq);
  mp = flagged(mp);
  mq = flagged(mq);
  pad_slice<DT, T, NB>(s, g, xp, xq);
  const int left = wave_left(s, g);
  float sum = phase1_sums<DT, T, NB, false, SKIP>(xp, xq, -mp, -mq, left);
  masked = __any(!(fabsf(sum) < INFINITY)) != 0;
  if (masked) sum = phase1_sums<DT, T, NB, true, SKIP>(xp, xq, -mp, -mq, left);
  // rows 0..3 of the lanes: S of the target row, U of the target row, S of the draft row, U of the draft row
  if ((lane & 15) == 0) sh.wave[wave].v[lane >> 4] = sum;
  if ((lane & 31) == 1) sh.wave[wave].m[lane >> 5] = lane < 32 ? mp : mq;
  lds_barrier();
  Lse f = lse_empty();
  if (wave != 0) return f;
  Lse tp = lse_empty(), tq = lse_empty();
  if (lane < W) record_rows(sh.wave[lane], tp, tq);
  f = fold_pair(tp, tq);
  f.m = flagged(f.m);       // (where every logit of the slice is masked, the lanes without a record have the largest reference)
  return f;
}

// The JS sum of the wavefront's share.  One element's term (see jsd_push, of which this is the ordinary form,
// four pairs at a time).  MASKED: as in phase 1.
template <int DT, int T, int NB, bool MASKED, bool SKIP>
__device__ __forceinline__ float phase2(const uint4 (&xp)[NB], const uint4 (&xq)[NB], float neg_cp, float neg_cq, float neg_dc, int left) {
  float acc[2] = {0.f, 0.f};
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    if (SKIP && j > 0 && j * T >= left) break;
#pragma unroll
    for (int half = 0; half < Elem<DT>::per_vec / 4; ++half) {
      float zp[4], zq[4], b[4], d[4], r[4], h[4], l[4];
      unpack4<DT, MASKED>(xp[j], half, zp);
      unpack4<DT, MASKED>(xq[j], half, zq);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        b[i] = max_raw(fma_log2e(zp[i], neg_cp), fma_log2e(zq[i], neg_cq));
        d[i] = fma_log2e(zq[i] - zp[i], neg_dc);
        if (MASKED) d[i] = fminf(fabsf(d[i]), 126.0f);      // (a NaN, from two masked logits, ends up there too)
      }
      ex2_group2(b, d, r);
#pragma unroll
      for (int i = 0; i < 4; ++i) h[i] = fmaf(r[i], 0.5f, 0.5f);
      lg2_group(h, l);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float t_log = fmaf(-2.0f, h[i] * l[i], r[i] * -fabsf(d[i]));
        const float d2 = d[i] * d[i];
        const float t_series = fmaf(d2, fmaf(d2, kJsC2, kJsC1), kJsC0) * d2 * h[i];
        acc[i & 1] = fmaf(b[i], fabsf(d[i]) < kJsSmall ? t_series : t_log, acc[i & 1]);
      }
    }
  }
  return acc[0] + acc[1];
}
// Rows whose normalisers lie far apart (rare, and not to set the kernel's register count).
template <int DT, int NB>
__device__ __forceinline__ float phase2_far(const uint4 (&xp)[NB], const uint4 (&xq)[NB], const JsNorm& n) {
  constexpr int EPV = Elem<DT>::per_vec;
  float acc = 0.f;
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    uint4 vp = xp[j], vq = xq[j];          // (opaque copies: see unpack4)
    asm volatile("" : "+v"(vp.x), "+v"(vp.y), "+v"(vp.z), "+v"(vp.w));
    asm volatile("" : "+v"(vq.x), "+v"(vq.y), "+v"(vq.z), "+v"(vq.w));
    float zp[EPV], zq[EPV];
    unpack<DT>(vp, zp);
    unpack<DT>(vq, zq);
#pragma unroll
    for (int e = 0; e < EPV; ++e) {
      jsd_push<true>(zp[e], zq[e], n, acc);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  return acc;
}

// The slice's record: the lower half of wavefront 0 holds the target row's share, the upper half the draft row's.
__device__ __forceinline__ void publish(const Workspace& ws, int pos, int s, const Lse& f) {
  const int lane = threadIdx.x & 63;
  uint64_t* w = ws.xchg + ((size_t)pos * kMaxSplit + s) * kXchgWords;
  float up = f.u, uq = f.u;
  swap32(up, uq);                         // up: the lower half's in every lane, uq: the upper half's
  // (lane 0 has the target row's share, lane 32 the draft row's, as where a record is kept: see row_sum16)
  auto put = [](uint64_t* p, uint64_t word) { __hip_atomic_store(p, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  if ((lane & 31) == 0) put(w + (lane >> 5), record_word(bits_of(f.m), lane == 0 ? sum_with_bit(f.s, f.u) : f.s));
  if (lane == 0) put(w + 2, record_word(bits_of(flagged(up)), uq));
}

// Wavefront 0: the rows' results and what phase 2 needs of them, from one slice record per lane.
__device__ __forceinline__ void fold_position(const Lse& tp, const Lse& tq, JsNorm& norm, RowResult (&row)[2], int& bad) {
  const RowResult mine = finish_row(fold_pair(tp, tq));   // (of the half's row)
  const int lane = threadIdx.x & 63;
  float lo_p = __int_as_float(__double2loint(mine.lse2)), lo_q = lo_p;
  float hi_p = __int_as_float(__double2hiint(mine.lse2)), hi_q = hi_p;
  float h_p = mine.H, h_q = mine.H, b_p = __int_as_float(mine.bad), b_q = b_p;
  swap32(lo_p, lo_q);
  swap32(hi_p, hi_q);
  swap32(h_p, h_q);
  swap32(b_p, b_q);
  const RowResult rp{__hiloint2double(__float_as_int(hi_p), __float_as_int(lo_p)), h_p, __float_as_int(b_p)};
  const RowResult rq{__hiloint2double(__float_as_int(hi_q), __float_as_int(lo_q)), h_q, __float_as_int(b_q)};
  if (lane == 0) {
    norm = js_norm(rp, rq);
    row[0] = rp;
    row[1] = rq;
    bad = rp.bad || rq.bad;
  }
}

template <int DT, int T, int NB, bool SKIP>
__global__ void __launch_bounds__(T, NB <= 4 ? 8 : 4)
k_stats_fused(RowMap map, FusedGeom g, Workspace ws, VerifyOut vout, HistArgs hist) {
  warm_kernargs<sizeof(RowMap) + sizeof(FusedGeom) + sizeof(Workspace) + sizeof(VerifyOut) + sizeof(HistArgs)>();
  constexpr int W = T / 64;
  __shared__ FusedShared<W> sh;
  const int s = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if ((int)blockIdx.y < g.hist_rows) {       // the first workgroups form the constants of the sequences' history lists
    __shared__ HistShared hsh;
    const int b = (int)(blockIdx.y * gridDim.x + blockIdx.x);
    if (b < hist.B) form_history<T>(hist, b, hsh);
    return;
  }
  const int pos = position_of_slot(map, (int)blockIdx.y - g.hist_rows);
  if (pos < 0) return;
  const RowRef rp = locate_row<DT>(map, 2 * pos), rq = locate_row<DT>(map, 2 * pos + 1);
  if (!rp.active) return;

  // the drafted token of the position (its two logits are looked up further down by one thread)
  const bool gathers = s == 0 && tid == 0 && vout.tok != nullptr;
  int x = -1;
  if (gathers) x = vout.tokens[pos];

  uint4 xp[NB], xq[NB];
  load_slice<DT, T, NB>(rp.ptr, rq.ptr, s, g, xp, xq);
  bool masked;
  const Lse mine = phase1<DT, T, NB, SKIP>(s, g, xp, xq, masked, sh);

  if (wave == 0) {
    const bool need = lane < g.S;
    bool ok = true;
    Lse tp = lse_empty(), tq = lse_empty();
    if (g.S > 1) {
      publish(ws, pos, s, mine);
      // every slice of the position, one per lane (this workgroup's own words come back the same way)
      const uint64_t* src = ws.xchg + ((size_t)pos * kMaxSplit + (need ? lane : 0)) * kXchgWords;
      uint64_t w0 = 0, w1 = 0, w2 = 0;
      bool there = !need;
      // The words are read past the caches, over the fabric that the logits come by: with a thousand workgroups waiting, their
      // reads are what holds up the records that they wait for.  So the first look comes after a nap (launch_stats_fused
      // says how long), and a later one asks for the records that are still missing alone.
      for (int i = 0; i < g.naps; ++i) __builtin_amdgcn_s_sleep(12);
      for (int polls = 0;;) {
        if (!there) {
          w0 = get_word(src + 0);
          w1 = get_word(src + 1);
          w2 = get_word(src + 2);
          there = (w0 & w1 & w2 & 1ull) != 0;
        }
        ok = __all(there) != 0;
        if (ok || ++polls > g.wait_polls) break;
        __builtin_amdgcn_s_sleep(4);
      }
      if (need) {
        const uint64_t w[kXchgWords] = {w0, w1, w2};
        const PairRecord r = unpack_pair(w);
        tp = Lse{r.mp, r.sp, r.up};
        tq = Lse{r.mq, r.sq, r.uq};
      }
    } else {                             // one slice per position: nothing travels through memory
      Lse a, b;
      split_halves(mine, a, b);
      if (lane == 0) {
        tp = a;
        tq = b;
      }
    }
    if (ok) fold_position(tp, tq, sh.norm, sh.row, sh.bad);
    if (lane == 0) sh.expired = ok ? 0 : 1;
  }
  lds_barrier();
  if (sh.expired) {                        // (uniform) the bounded wait ran out: every slice from memory
    auto keep = [&](int o, const Lse& f) {
      if (wave == 0 && (lane & 31) == 0) {
        const int row = lane >> 5;
        sh.redo[o].m[row] = f.m;
        sh.redo[o].v[2 * row] = f.s;
        sh.redo[o].v[2 * row + 1] = f.u;
      }
    };
    keep(s, mine);
    for (int o = 0; o < g.S; ++o) {
      if (o == s) continue;
      lds_barrier();                       // (sh.wave of the previous turn has been read)
      load_slice<DT, T, NB>(rp.ptr, rq.ptr, o, g, xp, xq);
      bool masked_o;
      keep(o, phase1<DT, T, NB, SKIP>(o, g, xp, xq, masked_o, sh));
    }
    lds_barrier();
    if (wave == 0) {
      Lse tp = lse_empty(), tq = lse_empty();
      if (lane < g.S) record_rows(sh.redo[lane], tp, tq);
      fold_position(tp, tq, sh.norm, sh.row, sh.bad);
    }
    // (the slice number goes through an opaque copy: otherwise the addresses of the loads at the top of the
    // kernel are kept in registers all the way down here, sixteen of them per thread)
    int s_again = s;
    asm volatile("" : "+s"(s_again));
    load_slice<DT, T, NB>(rp.ptr, rq.ptr, s_again, g, xp, xq);
    pad_slice<DT, T, NB>(s_again, g, xp, xq);
    lds_barrier();
  }

  const JsNorm n = sh.norm;
  const bool bad = sh.bad != 0;
  uint32_t zx_p = 0u, zx_q = 0u;
  if (gathers && x >= 0 && x < map.V) {
    zx_p = load_elem_bits<DT>(rp.ptr, x);
    zx_q = load_elem_bits<DT>(rq.ptr, x);
  }
  float acc = 0.f;
  if (!bad) {
    if (n.far) {
      acc = wave_sum_f(phase2_far<DT, NB>(xp, xq, n));
    } else {
      // (kept in vector registers: see device_common.h)
      float neg_cp = -n.cp, neg_cq = -n.cq, neg_dc = -n.dc_hi;
      asm volatile("" : "+v"(neg_cp), "+v"(neg_cq), "+v"(neg_dc));
      if (!masked) {
        acc = wave_sum_f(phase2<DT, T, NB, false, SKIP>(xp, xq, neg_cp, neg_cq, neg_dc, wave_left(s, g)));
        masked = !(fabsf(acc) < INFINITY);       // (the difference of two logits beyond the float range)
      }
      if (masked) acc = wave_sum_f(phase2<DT, T, NB, true, SKIP>(xp, xq, neg_cp, neg_cq, neg_dc, wave_left(s, g)));
    }
  }
  if (lane == 0) sh.acc[wave] = acc;
  lds_barrier();
  if (tid == 0) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < W; ++w) t += sh.acc[w];
    // partial sum of this slice: added up, corrected and turned into the distance by the decision kernel
    reinterpret_cast<float*>(&ws.part2[(size_t)pos * kMaxSplit + s])[0] = t;
    if (s == 0) {        // the position's rows and entropies, once
      const RowResult resp = sh.row[0], resq = sh.row[1];
      ws.rows[2 * pos] = resp;
      ws.rows[2 * pos + 1] = resq;
      if (vout.H_p) vout.H_p[pos] = resp.H;
      if (vout.H_q) vout.H_q[pos] = resq.H;
      if (vout.tok) vout.tok[pos] = make_float2(elem_from_bits<DT>(zx_p), elem_from_bits<DT>(zx_q));
    }
  }
}

}  // namespace

// Can the single-read kernel take this call, and with which tiling?  Rows of any alignment and of any length from one
// vector up, in at most kMaxSplit slices of at most eight vectors per thread and row.  Rows off a 16-byte boundary
// cost a cache line more per wavefront and load; the two-kernel path reads every logit twice, and such rows by
// element.  A round with this kernel against one with those two, bf16: 1 x 4 x 2001 15.5 / 19.8 us, 8 x 8 x 32003
// 23.6 / 28.2, 64 x 3 x 16001 23 / 33, 48 x 16 x 64001 78 / 209; float 1 x 4 x 32003 20.1 / 21.6, 48 x 16 x 64001
// 97 / 250: faster at all of the 48 odd shapes timed.  The statistics alone, from 9 to 1501 logits and 4 to 32000 positions,
// both types: 0.5 to 0.75 of the two kernels' time (1 x 4 x 9 4.1 / 8.1, 2000 x 16 x 101 float 105 / 161).
//
// Few positions leave most of the chip idle, and the kernel is then one chain of latencies in which a wavefront's own vectors
// and the eight wavefronts of a workgroup that share a compute unit stand one after the other: smaller workgroups, as long as
// each has a compute unit to itself (256), and as long as half of a position's hand-off slots stay free, for the decisions
// inside the token kernel (merges_decisions).  Whole calls (us), slices by V alone / up to 128 / 256 / 384 / 512 workgroups:
//   1 x 4 x 32000 bf16    16.6 / 14.0 / 14.1 / 14.0 / 14.0     16 x 4 x 16001             17.7 / 16.9 / 15.7 / 15.7 / 15.5
//   1 x 4 x 32000 float   14.6 / 13.1 / 13.1 / 13.1 / 13.2     4 x 8 x 50257              18.1 / 18.1 / 17.2 / 17.2 / 16.8
//   1 x 1 x 128256        17.0 / 14.7 / 14.7 / 14.7 / 14.7     1 x 20 x 128256            20.4 / 20.4 / 20.4 / 21.1 / 21.1
//   1 x 8 x 128256        17.1 / 16.1 / 15.0 / 15.0 / 15.0     16 x 6 x 32003 literal     19.4 / 19.4 / 19.4 / 19.8 / 19.8
//   4 x 4 x 128256        18.0 / 17.9 / 17.5 / 17.5 / 17.2     24 x 4 x 32003             20.1 / 20.3 / 20.1 / 20.9 / 20.7
// Beyond 256 some win 0.2 to 0.4 where their slices come to 512 workgroups, others lose as much or more.  Errors against 64 bits (rms, 60 rounds each), by V alone / up to 256: 1 x 4 x 32000 float
// entropies 4.5e-8 / 3.9e-8, distances 9.7e-8 / 1.03e-7; 1 x 8 x 128256 bf16 4.4e-8 / 4.2e-8, 1.34e-7 / 1.32e-7; 8 x 4 x 16001 4.9e-8
// / 4.9e-8, 1.69e-7 / 1.59e-7.
constexpr int kSmallGroups = 256, kSmallSplit = kMaxSplit / 2;
bool fused_plan(const RowMap& map, int dt, int* T_out, int* NB_out, int* S_out) {
  const int epv = dt == ADASD_BF16 ? 8 : 4;
  if (map.K <= 0 || map.V < epv) return false;
  const int nv = (map.V + epv - 1) / epv;
  int T = 512, NB = 4;
  while (T > 256 && nv <= (T / 2) * NB) T /= 2;                 // small vocabularies: smaller workgroups
  while (NB > 1 && nv <= T * (NB / 2)) NB /= 2;
  while (NB < 8 && (nv + T * NB - 1) / (T * NB) > kMaxSplit) NB *= 2;   // very large ones: more vectors per thread
  int S = (nv + T * NB - 1) / (T * NB);
  if (S > kMaxSplit) return false;
  while (NB <= 4 && (T > 256 || NB > 1)) {                      // few positions: more, smaller workgroups
    const int fewer = T * NB / 2, more = (nv + fewer - 1) / fewer;
    if (more > kSmallSplit || (int64_t)more * map.B * map.K > kSmallGroups) break;
    if (T > 256) T = 256;
    else NB /= 2;
    S = more;
  }
  *T_out = T;
  *NB_out = NB;
  *S_out = S;
  return true;
}

// Where the chip holds all workgroups of a round (1024 of 512 threads), or there is but one more set of them, a workgroup naps once
// (about 0.35 us, which the other slices need at least) before it first looks for their records; where there are more sets, three
// times, while other workgroups load.  Call times in us without a nap / with 1 / 2 / 3 / 4 (64 samples a list; half of the
// range of nine runs: 0.1 to 0.3 up to 1024 workgroups, 0.5 from there on, 1 to 2 from 4096 on):
//   1 x 4 x 32000 float (32 workgroups)   13.9 / 13.3 / 13.5 / 13.7 / 14.0     64 x 8 x 32000 float (2048)   44.0 / 44.1 / 44.3 / 44.4 / 44.7
//   1 x 8 x 128256 (256)                  15.6 / 15.0 / 15.1 / 15.4 / 15.7     36 x 8 x 128256 (2304)        64.1 / 64.5 / 64.4 / 63.6 / 62.9
//   16 x 4 x 16001 (256)                  15.8 / 15.7 / 16.0 / 16.3 / 16.6     40 x 8 x 128256 (2560)        67.9 / 68.2 / 67.7 / 67.6 / 67.0
//   16 x 8 x 128256 (1024)                36.2 / 36.2 / 36.1 / 36.5 / 36.7     8 x 20 x 128256 float (2560)  51.9 / 51.4 / 51.0 / 50.5 / 50.6
//   20 x 8 x 128256 (1280)                43.1 / 43.0 / 42.9 / 43.1 / 42.8     64 x 8 x 96000 (3072)         78.0 / 78.4 / 78.5 / 77.3 / 76.1
//   24 x 8 x 128256 (1536)                47.0 / 47.1 / 46.9 / 47.2 / 46.9     256 x 8 x 32000 (4096)        94.8 / 96.2 / 95.5 / 94.4 / 94.2
//   32 x 8 x 128256 (2048)                57.9 / 58.1 / 57.3 / 57.5 / 56.9     128 x 8 x 50257 float (7168)  104 / 103 / 103 / 103 / 102
//   64 x 8 x 64000 (2048)                 57.4 / 57.8 / 57.1 / 56.7 / 56.4     128 x 16 x 152064 (20480)     368 / 367 / 368 / 367 / 368
// At 2048 the three shapes do not agree, so the line is behind them; up to 1536, and from 7168 on, it makes no difference that
// shows but for the smallest rounds.
constexpr int kManyGroups = 2048;

hipError_t launch_stats_fused(const RowMap& map, int dt, int T, int NB, int S, int wait_polls,
                              const Workspace& ws, const VerifyOut& vout, const HistArgs& hist, hipStream_t st) {
  const int positions = map.B * map.K;
  if (positions <= 0) return hipSuccess;
  FusedGeom g;
  g.S = S;
  const int epv = dt == ADASD_BF16 ? 8 : 4;
  g.nv = (map.V + epv - 1) / epv;
  g.missing = g.nv * epv - map.V;
  g.last_byte = map.V * (16 / epv) - 16;
  // Equal slices: consecutive workgroups go to the eight dies in turn, so with eight slices a die gets the same
  // slice of every position, and one that is longer than the others sets the time (whole 128-byte lines all the same).
  g.chunk = ((g.nv + S - 1) / S + 7) / 8 * 8;
  if ((int64_t)g.chunk * (S - 1) >= g.nv || g.chunk > T * NB) g.chunk = (g.nv + S - 1) / S;
  g.wait_polls = wait_polls;
  g.naps = (int64_t)S * positions > kManyGroups ? 3 : 1;
  if (g.chunk > T * NB) return hipErrorInvalidValue;
  g.hist_rows = hist.rec ? (hist.B + S - 1) / S : 0;
  const dim3 grid(S, positions + g.hist_rows);
  const bool skip = NB > 1 && g.chunk <= NB * T - 64;     // the last wavefront has no lane in its last vector
#define ADASD_FUSED_CASE(DTV, TV, NBV) \
  if (dt == DTV && T == TV && NB == NBV) { \
    if (skip) launch_kernel((k_stats_fused<DTV, TV, NBV, (NBV > 1)>), grid, dim3(TV), st, map, g, ws, vout, hist); \
    else launch_kernel((k_stats_fused<DTV, TV, NBV, false>), grid, dim3(TV), st, map, g, ws, vout, hist); \
    return hipGetLastError(); \
  }
#define ADASD_FUSED_DT(DTV)      /* (what fused_plan can choose) */ \
  ADASD_FUSED_CASE(DTV, 256, 1) ADASD_FUSED_CASE(DTV, 256, 2) ADASD_FUSED_CASE(DTV, 256, 4) \
  ADASD_FUSED_CASE(DTV, 512, 4) ADASD_FUSED_CASE(DTV, 512, 8)
  ADASD_FUSED_DT(ADASD_BF16)
  ADASD_FUSED_DT(ADASD_F32)
#undef ADASD_FUSED_DT
#undef ADASD_FUSED_CASE
  return hipErrorInvalidValue;
}

}  // namespace adasd
