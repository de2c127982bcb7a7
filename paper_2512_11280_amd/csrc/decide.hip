// Acceptance decisions of one round (Section 2.1.3, Section 4.4 and the verification loop of
// Algorithm 1 of the paper) and the update of the adaptive state (Section 4.3; update lines).
#include "decide_device.h"
#include "internal.h"

namespace adasd {

namespace {

template <int DT, bool INLOOP, bool HIST, int T, int LP>
__global__ void __launch_bounds__(T) k_decide(DecideArgs a, UpdateArgs upd, Workspace ws) {
  warm_kernargs<sizeof(DecideArgs) + sizeof(UpdateArgs) + sizeof(Workspace)>();
  __shared__ DecideShared sh;
  const SequenceIn in = ask_sequence(a, upd, blockIdx.x, true);
  decide_sequence<DT, INLOOP, HIST, T, LP>(a, upd, ws, blockIdx.x, in, sh);
}

// Long histories: one workgroup per candidate position.  One workgroup, that of position 0 where it can be, does all the
// work of a sequence whose lists are still short and the others leave at once, so with more workgroups than the
// chip holds at a time those of position 0 have to come first in dispatch order or they queue behind the
// idle ones: grid (sequences, k_max).  A launch that gives every workgroup a compute unit of its own
// measured 0.4 us faster the other way round (grid (k_max, sequences)); `seq_first` says which it is.
template <int DT, bool INLOOP, bool HIST>
__global__ void __launch_bounds__(kBlock) k_decide_wide(DecideArgs a, UpdateArgs upd, Workspace ws, int seq_first) {
  warm_kernargs<sizeof(DecideArgs) + sizeof(UpdateArgs) + sizeof(Workspace) + sizeof(int)>();
  __shared__ DecideShared sh;
  __shared__ WideShared wsh;
  const int b = seq_first ? blockIdx.x : blockIdx.y, pos = seq_first ? blockIdx.y : blockIdx.x;
  // The launch is sized for long lists (the host only knows their capacity); a sequence whose lists are
  // still short is cheaper in the one-workgroup form, so one of its workgroups takes that and the others leave.
  // All of them have to go by the same lengths, but the one that decides also applies the round, maybe before another one
  // has started.  With HIST the first workgroup decides, and one that finds lengths which the round may have taken past the
  // line looks up what they were (decide_position_wide).  Without, the one that arrives last decides, when all have read
  // them (nobody applies anything: the first one).
  const int n_long = min(max(max(a.nA[b], a.nR[b]), 0), a.cap);
  if (__builtin_expect(n_long < kWideMin, 0)) {
    if (HIST || upd.B == 0) {
      if (pos != 0) return;
    } else {
      __syncthreads();
      if (threadIdx.x == 0) {
        int32_t* ticket = &ws.ticket2[b * ticket_stride(a.map.B, kTicket2Len)];
        wsh.last = atomicAdd(ticket, 1) == a.map.K - 1;
        if (wsh.last) __hip_atomic_store(ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      __syncthreads();
      if (!wsh.last) return;
    }
    decide_sequence<DT, INLOOP, HIST, kBlock, 32>(a, upd, ws, b, ask_sequence(a, upd, b, true), sh);
    return;
  }
  decide_position_wide<DT, INLOOP, HIST>(a, upd, ws, ws.pos_rec, b, pos, sh, wsh);
}

// ---------------------------------------------------------------------------------------------
// Update step: one wavefront per sequence, one lane per candidate position (k_max <= 64).  Every lane
// reads its position's distance at once; accepted positions that pass the open-interval filter are
// appended in position order (rank = number of passing positions before it, from a ballot).
// ---------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(64) k_update(UpdateArgs a) {
  warm_kernargs<sizeof(UpdateArgs)>();
  const int b = blockIdx.x;
  int kb = a.K;
  if (a.draft_len) kb = min(max(a.draft_len[b], 0), a.K);
  const int r = min(max(a.n_accept[b], 0), kb);
  update_sequence(a, b, threadIdx.x, r, kb);
}

__global__ void __launch_bounds__(64) k_state_init(UpdateArgs a) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= a.B) return;
  a.T_G[b] = 0.f;
  a.ent_sum[b] = 0.0;
  a.ent_cnt[b] = 0;
  a.nA[b] = 0;
  a.nR[b] = 0;
  if (a.mom)
    for (int x = 0; x < 4; ++x) a.mom[4 * b + x] = 0.0;
}

// Running sums of both lists of one sequence from scratch (one workgroup per sequence).
__global__ void __launch_bounds__(kBlock) k_state_refresh(UpdateArgs a) {
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nA = min(max(a.nA[b], 0), a.cap), nR = min(max(a.nR[b], 0), a.cap);
  const float* LA = a.LA + (size_t)b * a.cap;
  const float* LR = a.LR + (size_t)b * a.cap;
  const double cA = nA > 0 ? (double)LA[0] : 0.0, cR = nR > 0 ? (double)LR[0] : 0.0;
  double m[4] = {0.0, 0.0, 0.0, 0.0};
  for (int j = tid; j < nA; j += kBlock) {
    const double e = (double)LA[j] - cA;
    m[0] += e;
    m[1] += e * e;
  }
  for (int j = tid; j < nR; j += kBlock) {
    const double e = (double)LR[j] - cR;
    m[2] += e;
    m[3] += e * e;
  }
  __shared__ double sh[kWaves][4];
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    m[x] = wave_sum_d(m[x]);
  }
  if (lane == 0)
    for (int x = 0; x < 4; ++x) sh[wave][x] = m[x];
  __syncthreads();
  if (tid < 4) a.mom[4 * b + tid] = (sh[0][tid] + sh[1][tid]) + (sh[2][tid] + sh[3][tid]);
}

__global__ void __launch_bounds__(256) k_zero(uint32_t* p, size_t n) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = 0u;
}

}  // namespace

hipError_t launch_decide(const DecideArgs& a, const UpdateArgs& upd, const Workspace& ws, hipStream_t st) {
  if (a.map.B <= 0) return hipSuccess;
  const dim3 block(kBlock);
  if (a.cap >= kWideCap && a.map.K > 0 && !a.relaxed_off && a.LA && a.LR && a.nA && a.nR) {
    const int lead = a.map.B * a.map.K > 256 ? 1 : 0;   // (256 compute units)
    const dim3 grid(lead ? a.map.B : a.map.K, lead ? a.map.K : a.map.B);
#define ADASD_WIDE_CASE(DTV, INLOOPV, HISTV) \
    if (a.dt == DTV && (a.list_update != 0) == INLOOPV && (a.hist != nullptr) == HISTV) \
      launch_kernel((k_decide_wide<DTV, INLOOPV, HISTV>), grid, block, st, a, upd, ws, lead);
#define ADASD_WIDE_DT(DTV) \
    ADASD_WIDE_CASE(DTV, false, false) ADASD_WIDE_CASE(DTV, false, true) ADASD_WIDE_CASE(DTV, true, false) ADASD_WIDE_CASE(DTV, true, true)
    ADASD_WIDE_DT(ADASD_BF16)
    ADASD_WIDE_DT(ADASD_F32)
#undef ADASD_WIDE_DT
#undef ADASD_WIDE_CASE
    return hipGetLastError();
  }
  const dim3 grid(a.map.B);
  // The kernel is one chain of latencies, and each turn of the positions is the same chain over again: one turn up to
  // 16 positions with a wavefront each (a list per half: both at once), and beyond that half a wavefront to a position, which
  // takes 32 in a turn.  Kernel (us), a wavefront / half a wavefront (in as many groups up to 16), 32 sequences: k = 8, lists of
  // 64 6.1 / 6.0, 256 6.5 / 6.9, 448 7.5 / 8.5; k = 12 6.6 / 6.5, 7.0 / 7.3, 7.9 / 8.8; k = 20 7.9 / 7.6, 8.6 / 8.7, 10.2 / 10.8;
  // k = 40 11.8 / 9.6, 13.2 / 11.1, 16.1 / 13.9.  Fewer threads and more turns: k = 16 with 8 wavefronts 8.4, 9.1, 10.6 where 16 take
  // 7.2, 7.8, 8.8.
  const int LP = a.map.K > 16 ? 32 : 64, T = a.map.K <= 4 ? 256 : a.map.K <= 8 ? 512 : 1024;
#define ADASD_DECIDE_CASE(DTV, INLOOPV, HISTV, TV, LPV) \
  if (a.dt == DTV && (a.list_update != 0) == INLOOPV && (a.hist != nullptr) == HISTV && T == TV && LP == LPV) \
    launch_kernel((k_decide<DTV, INLOOPV, HISTV, TV, LPV>), grid, dim3(TV), st, a, upd, ws);
#define ADASD_DECIDE_T(DTV, INLOOPV, HISTV) \
  ADASD_DECIDE_CASE(DTV, INLOOPV, HISTV, 256, 64) ADASD_DECIDE_CASE(DTV, INLOOPV, HISTV, 512, 64) \
  ADASD_DECIDE_CASE(DTV, INLOOPV, HISTV, 1024, 64) ADASD_DECIDE_CASE(DTV, INLOOPV, HISTV, 1024, 32)
#define ADASD_DECIDE_DT(DTV) \
  ADASD_DECIDE_T(DTV, false, false) ADASD_DECIDE_T(DTV, false, true) ADASD_DECIDE_T(DTV, true, false) ADASD_DECIDE_T(DTV, true, true)
  ADASD_DECIDE_DT(ADASD_BF16)
  ADASD_DECIDE_DT(ADASD_F32)
#undef ADASD_DECIDE_DT
#undef ADASD_DECIDE_T
#undef ADASD_DECIDE_CASE
  return hipGetLastError();
}

hipError_t launch_update(const UpdateArgs& a, hipStream_t st) {
  if (a.B <= 0) return hipSuccess;
  launch_kernel(k_update, dim3(a.B), dim3(64), st, a);
  return hipGetLastError();
}

hipError_t launch_state_init(const UpdateArgs& a, hipStream_t st) {
  if (a.B <= 0) return hipSuccess;
  launch_kernel(k_state_init, dim3((a.B + 63) / 64), dim3(64), st, a);
  return hipGetLastError();
}

hipError_t launch_state_refresh(const UpdateArgs& a, hipStream_t st) {
  if (a.B <= 0 || !a.mom) return hipSuccess;
  launch_kernel(k_state_refresh, dim3(a.B), dim3(kBlock), st, a);
  return hipGetLastError();
}

hipError_t launch_zero(void* p, size_t bytes, hipStream_t st) {
  const size_t n = bytes / 4;
  if (n == 0) return hipSuccess;
  int blocks = (int)((n + 255) / 256);
  if (blocks > 1024) blocks = 1024;
  launch_kernel(k_zero, dim3(blocks), dim3(256), st, (uint32_t*)p, n);
  return hipGetLastError();
}

}  // namespace adasd
