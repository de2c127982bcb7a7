"""Rows at rest are not read (include/adasd.h): the drafting kernel itself, compiled for the CPU and run thread by thread over rows
that are not active and whose logits are not there at all (pages without access: a read ends the process that runs it).
A row at rest needs nothing of the other lanes, so everything that goes across lanes ends the process too.  (Not optimised: a load
whose value is not used then stays where the source has it.)"""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2512_11280_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"

SHIM = r"""
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <initializer_list>
using std::max; using std::min; using std::isnan;
#define __device__
#define __host__
#define __global__
#define __shared__ static
#define __forceinline__ inline
#define __launch_bounds__(...)
struct uint4 { uint32_t x, y, z, w; };
struct float4 { float x, y, z, w; };
struct float2 { float x, y; };
inline uint4 make_uint4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) { return {x, y, z, w}; }
struct dim3 { unsigned x, y, z; dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {} };
typedef int hipError_t; typedef void* hipStream_t; typedef void* hipEvent_t;
enum { hipSuccess = 0 };
inline int hipGetLastError() { return 0; }
#define hipLaunchKernelGGL(...) std::abort()
#define hipExtLaunchKernelGGL(...) std::abort()
inline dim3 threadIdx, blockIdx;
template <class T> T across_lanes(T) { std::abort(); }
#define __syncthreads() std::abort()
#define __any(x) across_lanes((int)(x))
#define __all(x) across_lanes((int)(x))
#define __ballot(x) across_lanes((unsigned long long)(x))
#define __shfl_xor(x, off) across_lanes(x)
#define __ffsll(x) __builtin_ffsll(x)
#define __popcll(x) __builtin_popcountll(x)
#define __builtin_amdgcn_readlane(x, l) across_lanes((int)(x))
#define __builtin_amdgcn_update_dpp(o, x, ...) across_lanes((int)(x))
struct Pair { uint32_t v[2]; uint32_t operator[](int i) const { return v[i]; } };
#define __builtin_amdgcn_permlane16_swap(a, b, ...) across_lanes(Pair{})
#define __builtin_amdgcn_permlane32_swap(a, b, ...) across_lanes(Pair{})
#define __builtin_amdgcn_readfirstlane(x) ((int)(x))      /* (of what is the same in every lane) */
#define __builtin_amdgcn_kernarg_segment_ptr() kernargs
inline char kernargs[4096];
#define __builtin_amdgcn_fence(...)
#define __builtin_amdgcn_s_waitcnt(x)
#define __builtin_amdgcn_exp2f(x) exp2f(x)
#define __builtin_amdgcn_logf(x) log2f(x)
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __builtin_amdgcn_fmed3f(a, b, c) fmaxf(fminf(a, b), fminf(fmaxf(a, b), c))
#define __builtin_amdgcn_bitop3_b32(a, b, c, t) ((a) ^ (b) ^ (c))
inline uint32_t __float_as_uint(float f) { uint32_t u; __builtin_memcpy(&u, &f, 4); return u; }
inline float __uint_as_float(uint32_t u) { float f; __builtin_memcpy(&f, &u, 4); return f; }
inline int __float_as_int(float f) { return (int)__float_as_uint(f); }
inline float __int_as_float(int i) { return __uint_as_float((uint32_t)i); }
template <class T> T atomicAdd(T* p, T v) { T o = *p; *p += v; return o; }
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __HIP_MEMORY_SCOPE_WORKGROUP 0
#define __HIP_MEMORY_SCOPE_WAVEFRONT 0
#define __hip_atomic_load(p, o, s) (*(p))
#define __hip_atomic_store(p, v, o, s) (*(p) = (v))
#define __hip_atomic_fetch_add(p, v, o, s) atomicAdd(p, v)
#define __hip_atomic_compare_exchange_strong(...) across_lanes(false)
"""

MAIN = r"""
#include "draft.hip"
#include <sys/mman.h>
#include <cstdio>
using namespace adasd;
bool adasd::profile_take_events(hipEvent_t*, hipEvent_t*) { return false; }
template <int DT, bool DRAW, bool PRUNE> int rows_at_rest(const char* nothing, int V) {
  const int B = 3, S = 2, chunk = sampling::slice_chunk(vectors_of<DT>(V), S);
  uint8_t active[B] = {0, 0, 0}, stop[B] = {7, 7, 7};
  float T_G[B] = {1.f, 2.f, 3.f}, H[B] = {7.f, 7.f, 7.f};
  int32_t token[B] = {7, 7, 7};
  uint32_t status[B] = {7, 7, 7};
  RowMap map{};
  map.base[0] = nothing;
  map.seq_stride[0] = V;
  map.active = active;
  map.B = B;
  map.V = V;
  const DraftOut dout{T_G, H, stop, 0, kWaits};
  const DraftDraw dr{1u, 2u, nullptr, nullptr, 3u, 0u, token, status};
  for (unsigned b = 0; b < (unsigned)B; ++b)
    for (unsigned s = 0; s < (unsigned)S; ++s)
      for (unsigned t = 0; t < (unsigned)kBlock; ++t) {
        blockIdx = dim3(s, b);
        threadIdx = dim3(t);
        k_draft<DT, DRAW, PRUNE>(map, S, chunk, Workspace{}, dout, dr);
      }
  for (int b = 0; b < B; ++b)
    if (H[b] != 0.f || stop[b] != 0 || (DRAW && (token[b] != -1 || status[b] != 0))) return 1;
  return 0;
}
int main() {
  const char* nothing = (const char*)mmap(nullptr, 1 << 20, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
  if (nothing == MAP_FAILED) return 2;
  int wrong = 0;
  for (int V : {5000, 5003}) {
    wrong |= rows_at_rest<ADASD_BF16, false, false>(nothing, V) | rows_at_rest<ADASD_F32, false, false>(nothing, V);
    wrong |= rows_at_rest<ADASD_BF16, true, false>(nothing, V) | rows_at_rest<ADASD_F32, true, false>(nothing, V);
    wrong |= rows_at_rest<ADASD_BF16, true, true>(nothing, V) | rows_at_rest<ADASD_F32, true, true>(nothing, V);
  }
  return wrong;
}
"""


def _without_asm(text):
    """The source with its assembler statements (issue order, and instructions that no thread of a row at rest gets to) taken out."""
    out, at = [], 0
    for m in re.finditer(r"\basm\s*(volatile)?\s*\(", text):
        if m.start() < at:
            continue
        depth, end, quoted = 1, m.end(), False
        while depth:
            c = text[end]
            quoted ^= c == '"' and text[end - 1] != "\\"
            depth += 0 if quoted else (c == "(") - (c == ")")
            end += 1
        out.append(text[at:m.start()])
        at = end
    return "".join(out) + text[at:]


@pytest.mark.skipif(not os.path.exists(CLANG), reason="needs ROCm's clang")
def test_rows_at_rest_are_not_read(tmp_path):
    for name in ("device_common.h", "records.h", "noise_series.h", "internal.h", "sample_device.h", "stats_device.h", "draft.hip"):
        with open(os.path.join(CSRC, name)) as f:
            (tmp_path / name).write_text(_without_asm(f.read()).replace('"../../include/adasd.h"', '"adasd.h"'))
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(SHIM)
    (tmp_path / "hip" / "hip_ext.h").write_text("#pragma once\n")
    (tmp_path / "main.cpp").write_text(MAIN)
    cmd = [CLANG, "-O0", "-std=c++17", "-w", "-I", str(tmp_path), "-I", os.path.join(ROOT, "include"), str(tmp_path / "main.cpp"),
           "-o", str(tmp_path / "rows")]
    built = subprocess.run(cmd, capture_output=True, text=True)
    assert built.returncode == 0, built.stderr
    assert subprocess.run([str(tmp_path / "rows")], timeout=60).returncode == 0
