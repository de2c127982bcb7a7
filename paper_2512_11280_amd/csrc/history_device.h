// Device code of the history lists (Section 4.4 of the paper): reductions in double precision, the kernel constants of a list,
// and their formation for a sequence ahead of its decisions.
#pragma once
#include "internal.h"

namespace adasd {

// ---- reductions over half a wavefront (32 lanes) in double precision: rotations inside the rows of
// 16 lanes on the two 32-bit halves, then one exchange between the two rows.  All 32 lanes get the result.
template <int CTRL> __device__ __forceinline__ double dpp_rot_d(double v) {
  const int lo = __double2loint(v), hi = __double2hiint(v);
  return __hiloint2double(__builtin_amdgcn_update_dpp(0, hi, CTRL, 0xf, 0xf, false),
                          __builtin_amdgcn_update_dpp(0, lo, CTRL, 0xf, 0xf, false));
}
// swap16 / swap32 (device_common.h) of the two halves of a double: of two copies of a value, the first becomes that of the even
// rows (the lower half), the second that of the odd rows (the upper half).
__device__ __forceinline__ void swap_rows(double& x, double& y) {
  float xl = __int_as_float(__double2loint(x)), xh = __int_as_float(__double2hiint(x));
  float yl = __int_as_float(__double2loint(y)), yh = __int_as_float(__double2hiint(y));
  swap16(xl, yl);
  swap16(xh, yh);
  x = __hiloint2double(__float_as_int(xh), __float_as_int(xl));
  y = __hiloint2double(__float_as_int(yh), __float_as_int(yl));
}
__device__ __forceinline__ void swap_halves(double& x, double& y) {
  float xl = __int_as_float(__double2loint(x)), xh = __int_as_float(__double2hiint(x));
  float yl = __int_as_float(__double2loint(y)), yh = __int_as_float(__double2hiint(y));
  swap32(xl, yl);
  swap32(xh, yh);
  x = __hiloint2double(__float_as_int(xh), __float_as_int(xl));
  y = __hiloint2double(__float_as_int(yh), __float_as_int(yl));
}
__device__ __forceinline__ double half_sum_d(double v) {
  v += dpp_rot_d<0x121>(v);
  v += dpp_rot_d<0x122>(v);
  v += dpp_rot_d<0x124>(v);
  v += dpp_rot_d<0x128>(v);
  double w = v;
  swap_rows(v, w);
  return v + w;
}
__device__ __forceinline__ double wave_sum_d(double v) {       // over the whole wavefront
  v = half_sum_d(v);
  double w = v;
  swap_halves(v, w);
  return v + w;
}
__device__ __forceinline__ double half_max_d(double v) {
  v = fmax(v, dpp_rot_d<0x121>(v));
  v = fmax(v, dpp_rot_d<0x122>(v));
  v = fmax(v, dpp_rot_d<0x124>(v));
  v = fmax(v, dpp_rot_d<0x128>(v));
  double w = v;
  swap_rows(v, w);
  return fmax(v, w);
}

struct Kde {
  double scale;    // log2(e) / (2 h^2): a kernel is 2 to the minus scale * (d - x)^2
  double log_norm; // log2(n h sqrt(2 pi)) - log2 prior  (subtracted from the log2 of the kernel sum)
};

// Gaussian-kernel constants of a history list from its shifted moments (sum and sum of squares of
// x - shift): sample variance with n-1, the bandwidth rule, the list-size prior.
__device__ inline bool kde_constants(double s1, double s2, int n, int n_other, int bw_rule, Kde* out) {
  const double var = (s2 - s1 * s1 / (double)n) / (double)(n - 1);
  if (!(var > 0.0)) return false;
  // x^(1/5) through the hardware exp2 / log2 (relative error about 1e-7: far inside what the
  // posterior's tolerance asks of the bandwidth)
  const float base = bw_rule == 1 ? 1.0f / (float)n : 4.0f / (3.0f * (float)n);
  const double factor = (double)ex2((float)(0.2 * log2_acc(base)));
  const double h = factor * sqrt(var);
  out->scale = 1.44269504088896340736 / (2.0 * h * h);
  const float prior = (float)n / (float)(n + n_other);
  out->log_norm = log2_acc((float)((double)n * h * 2.50662827463100050242)) - log2_acc(prior);
  return true;
}

// What the decisions of a sequence need to know of its lists beside the samples: formed by a workgroup of the statistics
// launch, beside the statistics, so that it does not stand in the chain of latencies of the decision kernel.
struct HistRecord {
  double c[2], s1[2], s2[2];     // accepted list, rejected list: first sample, sums of x - c and of its square
  Kde k[2];
  int32_t ok[2];                 // the constants hold: enough samples, and spread
  int32_t n[2];                  // the lengths, as the round finds them (the state's own words change while the decisions run)
};
static_assert(sizeof(HistRecord) <= 2 * kMaxSplit * sizeof(float4), "one record per position fits the region of the two-kernel path's partial sums");

struct HistShared {
  double m[8][4];
};
// One workgroup of T threads (at most 512).  Lists of more than kSumsMin samples have their sums in the state.
// A list costs three latencies (length, first sample and samples, the reduction) and some 200 instructions in double
// precision; in the decision kernel that stood in the chain of every wavefront.  Here it is one workgroup among
// those of the statistics, and the first one: its time does not show (statistics of 1 x 4 x 32000 6.1 us either way,
// 32 x 8 x 128256 39.3), and the decisions lose 0.5 to 1.5 us with short lists and 1.5 to 3 with long ones (kernel, 32
// sequences, k = 8: lists of 16 8.6 -> 6.4 us, 448 10.3 -> 8.3, 1024 11.1 -> 8.9, 4096 10.4 -> 8.6).
template <int T>
__device__ __forceinline__ void form_history(const HistArgs& h, int b, HistShared& sh) {
  constexpr int W = T / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nA = min(max(scalar_load(h.nA + b), 0), h.cap), nR = min(max(scalar_load(h.nR + b), 0), h.cap);
  const float* L[2] = {h.LA + (size_t)b * h.cap, h.LR + (size_t)b * h.cap};
  const int n[2] = {nA, nR};
  double c[2], m[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    c[q] = n[q] > 0 ? (double)L[q][0] : 0.0;
    if (h.mom && n[q] > kSumsMin) continue;           // (uniform)
#pragma unroll 1
    for (int base = 0; base < n[q]; base += 4 * T) {
      float x[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) x[u] = L[q][min(base + tid + u * T, n[q] - 1)];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const double e = base + tid + u * T < n[q] ? (double)x[u] - c[q] : 0.0;
        m[2 * q] += e;
        m[2 * q + 1] += e * e;
      }
    }
  }
#pragma unroll
  for (int x = 0; x < 4; ++x) m[x] = wave_sum_d(m[x]);
  if (lane == 0) {
#pragma unroll
    for (int x = 0; x < 4; ++x) sh.m[wave][x] = m[x];
  }
  __syncthreads();
  if (tid >= 64 || (lane & 31) != 0) return;
  // lane 0 finishes the accepted list, lane 32 the rejected one
  const int q = lane >> 5;
  double s1 = 0.0, s2 = 0.0;
#pragma unroll
  for (int v = 0; v < W; ++v) {
    s1 += sh.m[v][2 * q];
    s2 += sh.m[v][2 * q + 1];
  }
  const int mine = q ? nR : nA, other = q ? nA : nR;
  if (h.mom && mine > kSumsMin) {
    s1 = h.mom[4 * b + 2 * q];
    s2 = h.mom[4 * b + 2 * q + 1];
  }
  HistRecord* rec = h.rec + b;
  Kde k{0.0, 0.0};
  rec->n[q] = mine;
  rec->ok[q] = mine >= 2 && kde_constants(s1, s2, mine, other, h.bw_rule, &k);
  rec->c[q] = q ? c[1] : c[0];
  rec->s1[q] = s1;
  rec->s2[q] = s2;
  rec->k[q] = k;
}

}  // namespace adasd
