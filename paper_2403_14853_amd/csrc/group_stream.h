// Lane groups (gfx950, wave64): what the run-streaming kernels (run_stream.h) share.  A group of LPG consecutive lanes
// spans one dense row slice; G = 64 / LPG groups of a wavefront work on G stored entries at a time.
#pragma once
#include "block_scan.h"
#include "row_stream.h"

namespace isp_dev {

// Partition limits these kernels' LDS tables are sized for (csr_build clamps its parameters to them).
constexpr int GS_MAX_ENT = 768;    // nonzeros per item:  block_cost - 1 + hub_t  or  seg_len
constexpr int GS_MAX_ROWS = 256;   // rows per item: block_cost

typedef unsigned short gs_u16;

// Sum over the LPG consecutive lanes of a group, result in every lane of the group.  Lane
// exchanges inside 16 lanes are DPP modifiers (no LDS traffic); xor 16 is a ds_swizzle, xor 32 a
// bpermute.
template <int LPG>
__device__ inline float group_allreduce(float v) {
  // quad_perm [1,0,3,2] and [2,3,0,1]: xor 1, xor 2
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, true));
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, true));
  if constexpr (LPG >= 8)  // row_half_mirror (reverse within 8 lanes): pairs the two quads of an 8-lane half
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xF, 0xF, true));
  if constexpr (LPG >= 16)  // row_mirror (reverse within 16 lanes)
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x140, 0xF, 0xF, true));
  if constexpr (LPG >= 32)  // swap halves of 32 lanes: swizzle bit mode, xor mask 0x10
    v += __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), 0x401F));
  if constexpr (LPG >= 64) v += __shfl_xor(v, 32);
  return v;
}

// Four sums of LPG lanes at once: of a value per lane and step (p0 ... p3) each lane gets the group's total of step
// group_step<LPG>(lane), and of the lanes with the same total group_step_owner<LPG> says one.  A stage halves the
// values while there are several (a lane keeps one and hands the other to its partner), so four totals take 9 to 11 instructions
// where four sums after one another take 8 (4 lanes) to 24 (64), and what is computed from a total is computed once,
// not in every lane of the group.
template <int LPG>
__device__ __forceinline__ int group_step(int lane) {
  if constexpr (LPG == 4) return (lane >> 1 & 1) | (lane << 1 & 2);
  else if constexpr (LPG == 8) return (lane >> 2 & 1) | (lane & 2);
  else if constexpr (LPG == 16) return (lane >> 3 & 1) | (lane >> 1 & 2);
  else if constexpr (LPG == 32) return (lane >> 4 & 1) | (lane >> 2 & 2);
  else return (lane >> 5 & 1) | (lane >> 3 & 2);
}
template <int LPG>
__device__ __forceinline__ bool group_step_owner(int lane) { return (lane & (LPG / 4 - 1)) == 0; }

template <int CTRL>
__device__ __forceinline__ float dpp_of(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
// lanes with `up` keep b and get their partner's b, the others a; CTRL moves a value to the partner
template <int CTRL>
__device__ __forceinline__ float pair_sum(float a, float b, bool up) { return (up ? b : a) + dpp_of<CTRL>(up ? a : b); }
// (exchanges between rows of 16 and 32 lanes: one instruction hands b's even rows to a and a's odd rows to b)
__device__ __forceinline__ float pair_sum_16(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float pair_sum_32(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_HALF_MIRROR = 0x141, DPP_ROR8 = 0x128;  // (mirror: the other quad of 8 lanes)

template <int LPG>
__device__ __forceinline__ float group_sum_steps(float p0, float p1, float p2, float p3, int lane) {
  float v;
  if constexpr (LPG == 4) {
    return pair_sum<DPP_XOR1>(pair_sum<DPP_XOR2>(p0, p1, lane & 2), pair_sum<DPP_XOR2>(p2, p3, lane & 2), lane & 1);
  } else if constexpr (LPG == 8) {
    v = pair_sum<DPP_XOR2>(pair_sum<DPP_HALF_MIRROR>(p0, p1, lane & 4), pair_sum<DPP_HALF_MIRROR>(p2, p3, lane & 4), lane & 2);
    return v + dpp_of<DPP_XOR1>(v);
  } else if constexpr (LPG == 16) {
    v = pair_sum<DPP_HALF_MIRROR>(pair_sum<DPP_ROR8>(p0, p1, lane & 8), pair_sum<DPP_ROR8>(p2, p3, lane & 8), lane & 4);
  } else if constexpr (LPG == 32) {
    v = pair_sum<DPP_ROR8>(pair_sum_16(p0, p1), pair_sum_16(p2, p3), lane & 8);
    v += dpp_of<DPP_HALF_MIRROR>(v);
  } else {
    v = pair_sum_16(pair_sum_32(p0, p1), pair_sum_32(p2, p3));
    v += dpp_of<DPP_ROR8>(v);
    v += dpp_of<DPP_HALF_MIRROR>(v);
  }
  v += dpp_of<DPP_XOR1>(v);
  return v + dpp_of<DPP_XOR2>(v);
}
// of four steps' values, step group_step(lane)'s
template <int LPG>
__device__ __forceinline__ float group_step_value(float p0, float p1, float p2, float p3, int lane) {
  const int s = group_step<LPG>(lane);
  const float lo = s & 1 ? p1 : p0, hi = s & 1 ? p3 : p2;
  return s & 2 ? hi : lo;
}

// Two sums of LPG lanes at once, 16 lanes and more: of a value per lane and step (p0, p1) half of the group's lanes get the total of the first, the
// others of the second, so that what is computed from a total is computed once for both; group_pair_split then hands both results
// to all lanes.  A pair of sums takes 6 instructions with 16 or 32 lanes and 9 with 64, where two sums take 8, 12 and 16, the latter with exchanges
// through LDS; every result handed back takes 3 more with 16 lanes and 2 with 32 or 64.  So 16 lanes gain by the shared evaluation of the
// edge function alone (two dot products and one or two results: 15 or 18 instead of 16, less one evaluation), more lanes by both.
template <int LPG>
__device__ __forceinline__ float group_pair_sum(float p0, float p1, int lane) {
  static_assert(LPG >= 16, "no policy pairs entries with fewer lanes");
  float v;
  if constexpr (LPG == 16) v = pair_sum<DPP_ROR8>(p0, p1, lane & 8);
  else if constexpr (LPG == 32) v = pair_sum_16(p0, p1);
  else {
    v = pair_sum_32(p0, p1);
    v = pair_sum_16(v, v);
  }
  if constexpr (LPG > 16) v += dpp_of<DPP_ROR8>(v);
  v += dpp_of<DPP_HALF_MIRROR>(v);
  v += dpp_of<DPP_XOR1>(v);
  return v + dpp_of<DPP_XOR2>(v);
}
template <int LPG>
__device__ __forceinline__ void group_pair_split(float v, int lane, float& v0, float& v1) {
  static_assert(LPG >= 16, "no policy pairs entries with fewer lanes");
  if constexpr (LPG == 16) {
    const bool up = lane & 8;
    const float other = dpp_of<DPP_ROR8>(v);
    v0 = up ? other : v;
    v1 = up ? v : other;
  } else if constexpr (LPG == 32) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v0 = __uint_as_float(r[0]);
    v1 = __uint_as_float(r[1]);
  } else {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v0 = __uint_as_float(r[0]);
    v1 = __uint_as_float(r[1]);
  }
}

// Sum W values per lane over the G = 64 / LPG groups (lanes with equal lane % LPG), leaving the sums spread over
// the groups instead of complete in one: a stage that pairs lanes `O` apart splits the values in two halves,
// each lane of a pair keeps one half and receives the partner's share of it, so the stages move W/2 + W/4 + ...
// values instead of W each.  Afterwards the lane holds, in v[0 .. R), R = max(1, W / G), the finished sums of
// its values idx0 .. idx0 + R (idx0 is returned).  With more groups than values (G > W) the last stages add
// single values both ways and the groups whose lane number has a bit of (64 / W - 1) & ~(LPG - 1) set hold
// copies: group_owner<LPG, W>(lane) says which lanes hold the ones to store.  The order of the additions is
// fixed, so results repeat bit for bit.
template <int O, int LPG, int N, int W>
__device__ inline void group_reduce_stage(float (&v)[W], int lane, int& idx0) {
  if constexpr (O >= LPG) {
    if constexpr (N > 1) {
      const bool up = (lane & O) != 0;
#pragma unroll
      for (int c = 0; c < N / 2; ++c) {
        const float send = up ? v[c] : v[c + N / 2];
        const float keep = up ? v[c + N / 2] : v[c];
        v[c] = keep + __shfl_xor(send, O);
      }
      idx0 += up ? N / 2 : 0;
      group_reduce_stage<O / 2, LPG, N / 2, W>(v, lane, idx0);
    } else {
      v[0] += __shfl_xor(v[0], O);
      group_reduce_stage<O / 2, LPG, 1, W>(v, lane, idx0);
    }
  }
}
template <int LPG, int W>
__device__ inline int group_reduce_scatter(float (&v)[W], int lane) {
  int idx0 = 0;
  group_reduce_stage<ISP_WAVE / 2, LPG, W, W>(v, lane, idx0);
  return idx0;
}
template <int LPG, int W>
__device__ inline bool group_owner(int lane) {
  return (lane & ((ISP_WAVE / W - 1) & ~(LPG - 1))) == 0;
}

}  // namespace isp_dev
