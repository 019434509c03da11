// Hub rows put together by the launch that computes their segments (gfx950, wave64).
//
// A hub row's segments leave partial rows, which k_*_fixup adds in a launch of its own.  That launch is some 3 us and a
// drained chip whatever it adds, a third of what SpMM takes on 100 k entries.  Here each segment counts itself in at its
// row's counter once its partial row is written, and the one that counts last adds the row's partial rows at once: every
// segment may be that one, and the sum is the same whichever it is, in the fix-up's own order (quarters of the segments,
// each in order, then the quarters in order), so calls that use the fix-up - aliases, the static scratch - give the same bits.
//
// The segments of a row run on several XCDs, whose L2s do not see each other's writes: partial rows are written and read
// past the L2s (sc1: at the device's scope), which costs these stores and loads nothing that the fix-up's did not pay, where a
// release and acquire of the whole L2 would write back and drop everything else in it.  The counter is an increment that
// wraps to zero at the row's number of segments: nothing has to be cleared between launches.
#pragma once
#include "hub_rule.h"
#include "row_stream.h"

namespace isp_dev {

// A segment's row: its partial rows [s0, s1) and its counter.
struct hub_ref {
  int h, s0, s1;
};

constexpr int HF_SC1 = 16;  // cache policy bit of the buffer instructions: device scope
typedef unsigned hf_u4 __attribute__((ext_vector_type(4)));
typedef unsigned hf_u2 __attribute__((ext_vector_type(2)));

// base: wave-uniform; byte offsets below 2^31
template <int N>
__device__ __forceinline__ void hf_store(float* base, unsigned byte, const float (&o)[N]) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(base, 0, 0x7fffffff, 0x00027000);
  if constexpr (N == 4) {
    const hf_u4 v = {__float_as_uint(o[0]), __float_as_uint(o[1]), __float_as_uint(o[2]), __float_as_uint(o[3])};
    __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)byte, 0, HF_SC1);
  } else if constexpr (N == 2) {
    const hf_u2 v = {__float_as_uint(o[0]), __float_as_uint(o[1])};
    __builtin_amdgcn_raw_buffer_store_b64(v, r, (int)byte, 0, HF_SC1);
  } else {
    static_assert(N == 1);
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(o[0]), r, (int)byte, 0, HF_SC1);
  }
}
__device__ __forceinline__ void hf_load(float* base, unsigned byte, float (&o)[4]) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(base, 0, 0x7fffffff, 0x00027000);
  const hf_u4 v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)byte, 0, HF_SC1);
  o[0] = __uint_as_float(v.x); o[1] = __uint_as_float(v.y); o[2] = __uint_as_float(v.z); o[3] = __uint_as_float(v.w);
}

// The whole wavefront, after its segment's partial row is stored with hf_store: is this the row's last segment?
__device__ __forceinline__ bool hf_last(const isp_view& A, const hub_ref& H, int slice, int lane) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the partial row has arrived where every XCD reads it
  const unsigned n = (unsigned)(H.s1 - H.s0);
  unsigned before = 0;
  if (lane == 0) before = atomicInc(A.hub_done + (int64_t)H.h * HF_STRIDE + slice, n - 1u);
  const bool last = (unsigned)__builtin_amdgcn_readfirstlane((int)before) == n - 1u;
  asm volatile("" ::: "memory");
  return last;
}

// The sum of the row's partial rows over this lane's 4 columns, which start at byte `byte` of a partial row; complete in the
// lanes of group 0.  LPG lanes to a group; groups 0 to 3 take a quarter each, fewer groups several.  FLIGHT loads in flight per lane.
template <int LPG, int FLIGHT>
__device__ __forceinline__ void hf_sum(const isp_view& A, const hub_ref& H, unsigned byte, int lane, float (&sum)[4]) {
  constexpr int G = ISP_WAVE / LPG;
  constexpr int GQ = G < 4 ? G : 4;   // groups at work
  constexpr int QL = 4 / GQ;          // quarters per group
  constexpr int U = FLIGHT / QL;      // partial rows of a quarter in flight
  float* base = A.partials + (int64_t)H.s0 * ISP_PARTIAL_TILE;
  const int n = H.s1 - H.s0, q = (n + 3) / 4;
  const int g = lane / LPG < GQ ? lane / LPG : GQ - 1;  // (idle groups repeat the last one)
  float acc[QL][4];
#pragma unroll
  for (int k = 0; k < QL; ++k)
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[k][v] = 0.f;
  for (int i = 0; i < q; i += U) {
    float t[QL][U][4];
#pragma unroll
    for (int k = 0; k < QL; ++k)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int s = (g * QL + k) * q + i + u;
        hf_load(base, (unsigned)(s < n ? s : n - 1) * (unsigned)(ISP_PARTIAL_TILE * 4) + byte, t[k][u]);
      }
#pragma unroll
    for (int k = 0; k < QL; ++k)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool on = i + u < q && (g * QL + k) * q + i + u < n;
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[k][v] += on ? t[k][u][v] : 0.f;
      }
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float p = __shfl(acc[w % QL][v], (w / QL) * LPG + lane % LPG);
      t = w == 0 ? p : t + p;
    }
    sum[v] = t;
  }
}

}  // namespace isp_dev
