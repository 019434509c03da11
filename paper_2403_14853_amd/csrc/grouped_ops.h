// Grouped kernels for the operations that need a whole dot product per nonzero (SDDMM and the
// FusedMM passes).  The work items and contiguous runs of run_stream.h; here a
// group of LPG lanes spans the full feature width (W * LPG >= d with W = 4 or 8 floats per lane, as one
// or two float4), so G = 64 / LPG dot products are reduced side by side with the same DPP
// instructions.  Two float4 per lane halve the lanes per dot product: a step covers twice the entries,
// with one lane-reduction stage and one evaluation of the edge function less per entry - these kernels
// keep the vector ALU busy, so instructions per entry count.  The row operand (U's row for SDDMM, x_i / g_i
// for FusedMM) is loaded once per hub segment, which is one row throughout.  In row blocks one float4 per
// lane loads it with a row's first step in a run and keeps it; two float4 load it with every step (an L1 hit
// after the first).
#pragma once
#include <type_traits>
#include "hub_finish.h"
#include "run_stream.h"

namespace isp_dev {

// Policy P:  NSRC gathered operands (rows picked by column index), NROW row operands (rows picked
// by the entry's matrix row); RING4 / RING8 steps in flight with one / two float4 per lane;
// args { src[NSRC], lds_[NSRC], rowop[NROW], ldr[NROW], out_entry };
// either edge<LPG>(args, a, src, rowop, acc, lane_on) accumulating into the row's result, or (PER_ENTRY)
// partial(src, rowop, lane_cols) returning the lane's share of a sum over the group, which times the entry's value is stored
// for the entry.
// A policy with PAIR_LPG has three steps in place of edge(): dots(x, r, lane_cols, p), the lane's shares of NDOT dot products (0:
// none are needed); scalars(t, s), what the edge function makes of their totals, NSCAL numbers; apply(a, s, x, acc).  Groups of PAIR_LPG
// lanes and more work on two entries at a time where the ring holds four: the totals share their reduction over the lanes and one evaluation
// of the edge function, whose exponential and reciprocal take as long as eight other instructions (from which width on that pays: with
// the policies).
// A policy with HAS_VAL2 = true also gets a second value per stored entry, args::val2[p] (a parallel array in
// the order of the matrix's entries; null = all ones), as an extra argument of edge().
// ADDR32: every byte offset into the gathered operands fits 32 bits and both factors of column * row pitch
// fit 24 bits (fused_offsets_fit_32 below), so a gather address is one full-rate 24-bit multiply-add on a
// scalar base pointer instead of a 64-bit multiply (three quarter-rate instructions).
// values may be null (every stored value is 1).
// A lane's float4 vectors: whether each lies inside the feature width, and its first column (0 when it does not,
// so that the lane still reads valid memory).  TAIL (a width that is no multiple of 4): the last vector of a row
// moves back to end with the last column; dup = how many of its leading columns belong to the vector before it
// and must not be counted twice in a dot product.
template <int NV, bool TAIL>
struct lane_cols {
  bool on[NV];
  int off[NV];
  int dup[NV];
};

template <class P, class = void>
struct policy_has_val2 : std::false_type {};
template <class P>
struct policy_has_val2<P, std::void_t<decltype(P::HAS_VAL2)>> : std::bool_constant<P::HAS_VAL2> {};

template <class P, class = void>
struct policy_in_steps : std::false_type {};
template <class P>
struct policy_in_steps<P, std::void_t<decltype(P::PAIR_LPG)>> : std::true_type {};
template <class P, int LPG, int RING>
constexpr bool policy_pairs() {
  if constexpr (policy_in_steps<P>::value) return P::NDOT > 0 && LPG >= P::PAIR_LPG && RING >= 4;
  else return false;
}

// FINISH: the launch puts hub rows together (hub_finish.h).
template <class P, int LPG, int W, bool ADDR32, bool TAIL, bool FINISH = false, class Lds>
__device__ inline void fused_grouped_item(const isp_view& A, const int64_t* __restrict__ indptr,
                                          const int32_t* __restrict__ indices, const float* __restrict__ values,
                                          const typename P::args& pa, int d, float* __restrict__ Y, int64_t ldy,
                                          Lds& lds, int k_lo = 0) {
  // k_lo: first feature column of this pass (only the per-entry policies run in column windows;
  // their partial dot products are then added up across passes)
  static_assert(W == 4 || W == 8, "one or two float4 per lane");
  constexpr int G = ISP_WAVE / LPG;
  constexpr int NV = W / 4;  // float4 vectors per lane: vector v covers columns [v * 4 * LPG, (v + 1) * 4 * LPG)
  constexpr int NSRC = P::NSRC, NROW = P::NROW;
  constexpr int RING = W == 4 ? P::RING4 : P::RING8;
  constexpr int CHUNK = RING % 4 == 0 ? 2 : 1;
  const int lane = threadIdx.x & (ISP_WAVE - 1);
  const int w = threadIdx.x >> 6;
  const int item = __builtin_amdgcn_readfirstlane((int)blockIdx.x * ISP_WAVES_PER_WG + w);
  if (item >= A.n_blocks + A.n_seg) return;
  const item_range it = locate_item(A, indptr, item);
  if (it.skip) return;
  auto& L = lds.w[w];
  const bool finish = FINISH && it.is_seg;
  hub_ref H{0, 0, 0};
  if (finish) H.h = A.seg_hub[it.row];
  const rn_run R = rn_prepare<G>(it, indptr, indices, values, nullptr, L, lane);
  if (finish) {
    H.s0 = A.hub_seg_ptr[H.h];
    H.s1 = A.hub_seg_ptr[H.h + 1];
  }

  const int g = lane / LPG, q = lane % LPG;
  lane_cols<NV, TAIL> lc;  // this lane's columns: in range?  offset of the first (0 when out of range)
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int col = k_lo + v * 4 * LPG + q * 4;
    lc.on[v] = col < d;
    lc.off[v] = lc.on[v] ? (TAIL && col + 4 > d ? d - 4 : col) : 0;
    lc.dup[v] = TAIL && lc.on[v] ? col - lc.off[v] : 0;
  }
  float acc[W], head[W];  // head: the end of a row that began in an earlier run
#pragma unroll
  for (int v = 0; v < W; ++v) acc[v] = head[v] = 0.f;
  auto store_to = [&](float* o, const float (&src)[W]) {  // this lane's columns of the output row at o
    float t[W];
#pragma unroll
    for (int v = 0; v < W; ++v) t[v] = src[v];
    if (P::ACCUMULATE) {  // (all of it is read before anything is written: a moved-back vector overlaps)
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        float old[4];
        load_vec<4>(o + lc.off[v], old);
#pragma unroll
        for (int c = 0; c < 4; ++c) t[4 * v + c] += old[c];
      }
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      float part[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) part[c] = t[4 * v + c];
      if (lc.on[v]) store_vec<4>(o + lc.off[v], part);
    }
  };
  auto store_row = [&](int row, const float (&src)[W]) { store_to(Y + row * ldy, src); };  // (of a row block)
  if (!P::PER_ENTRY && !P::ACCUMULATE)  // outputs of the empty rows
    for (int i = g; i < R.n_empty; i += G) store_row(L.dst[RN_EMPTY0 - i], acc);

  auto load_w = [&](const float* p, float (&dst)[W]) {  // this lane's columns of the row that starts at p
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      float t[4];
      load_vec<4>(p + lc.off[v], t);
#pragma unroll
      for (int c = 0; c < 4; ++c) dst[4 * v + c] = t[c];
    }
  };
  auto load_at = [&](const float* base, int64_t ld, int row, float (&dst)[W]) {
    if constexpr (ADDR32) {
      const unsigned off = __umul24((unsigned)row, (unsigned)ld * 4u);
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        float t[4];
        load_vec<4>(reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + (off + (unsigned)lc.off[v] * 4u)), t);
#pragma unroll
        for (int c = 0; c < 4; ++c) dst[4 * v + c] = t[c];
      }
    } else {
      load_w(base + (int64_t)row * ld, dst);
    }
  };

  // The row operand of a row's first step; the row's other steps all read one and the same line instead, which keeps
  // the number of loads per step fixed (exact wait counts) and the lines they touch few.
  constexpr bool FIRST_ONLY = W == 4;
  auto load_first = [&](const float* base, int64_t ld, int row, bool first, float (&dst)[W]) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      float t[4];
      if constexpr (!FIRST_ONLY) first = true;
      if constexpr (ADDR32) {
        const unsigned off = first ? __umul24((unsigned)row, (unsigned)ld * 4u) + (unsigned)lc.off[v] * 4u : 0u;
        load_vec<4>(reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + off), t);
      } else {
        load_vec<4>(base + (first ? (int64_t)row * ld + lc.off[v] : 0), t);
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) dst[4 * v + c] = t[c];
    }
  };

  bool carried = R.mid;  // the next row to end began in an earlier run
  bool ended = false;    // a row has ended in this run
  // PER_ENTRY: four steps' shares are summed over the group at a time.  A result is parked in its entry's LDS slot (the entry
  // has been read) and written out in one coalesced sweep when the item is done.
  float share[4] = {0.f, 0.f, 0.f, 0.f}, share_a[4] = {0.f, 0.f, 0.f, 0.f};
  auto park = [&](int s0, int n) {  // steps [s0, s0 + n) of the run
    const float val = group_step_value<LPG>(share_a[0], share_a[1], share_a[2], share_a[3], lane) *
                      group_sum_steps<LPG>(share[0], share[1], share[2], share[3], lane);
    const int k = group_step<LPG>(lane);
    if (group_step_owner<LPG>(lane) && k < n) L.ent[R.start + s0 + k].y = __float_as_int(val);
  };
  // SEG (a hub segment: one matrix row for the whole item): the row operand is loaded once and stays in
  // registers.  Row blocks issue a load with every step (load_first), FIRST_ONLY or not, which keeps their loop free
  // of row-change stalls.
  auto run = [&](auto seg_tag) {
    constexpr bool SEG = decltype(seg_tag)::value;
    constexpr int NR = SEG ? 0 : NROW;  // per-step row-operand registers
    float rS[NROW][W];
    if constexpr (SEG) {
#pragma unroll
      for (int k = 0; k < NROW; ++k) load_w(pa.rowop[k] + (int64_t)it.src_row * pa.ldr[k], rS[k]);
    }
    float x[RING][NSRC][W], r[RING][NR + 1][W], a2[RING];
    bool first = true;  // the step to take next is its row's first in this run
    bool firsts[RING];  // PER_ENTRY, where nothing else happens at row ends: the same, kept since the step was requested
    // two steps at a time, where that leaves another two in flight
    constexpr bool PAIRS = policy_pairs<P, LPG, RING>();
    float sc[2][2];  // (of the pair's steps, NSCAL each)
    auto pair = [&](auto u0) {
      if constexpr (PAIRS) {
        constexpr int U = decltype(u0)::value, ND = P::NDOT, NS = P::NSCAL;
        float p[2][ND], t[ND], o[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          if constexpr (!SEG) {
            if (firsts[U + k] || !FIRST_ONLY) {
#pragma unroll
              for (int j = 0; j < NROW; ++j)
#pragma unroll
                for (int v = 0; v < W; ++v) rS[j][v] = r[U + k][j < NR ? j : 0][v];
            }
          }
          P::template dots<W, TAIL>(x[U + k], rS, lc, p[k]);
#pragma unroll
          for (int j = 0; j < ND; ++j) asm volatile("" : "+v"(p[k][j]));  // (formed before the next step's row operand takes the registers)
        }
#pragma unroll
        for (int j = 0; j < ND; ++j) t[j] = group_pair_sum<LPG>(p[0][j], p[1][j], lane);
        P::scalars(t, o);
#pragma unroll
        for (int j = 0; j < NS; ++j) group_pair_split<LPG>(o[j], lane, sc[0][j], sc[1][j]);
      }
    };
    rn_stream<RING, !SEG && !P::PER_ENTRY, !SEG, CHUNK, PAIRS>(
        L, R,
        [&](int u, int c, int s, int row, bool in_first) {
#pragma unroll
          for (int k = 0; k < NSRC; ++k) load_at(pa.src[k], pa.lds_[k], c, x[u][k]);
          if constexpr (!SEG) {
#pragma unroll
            for (int k = 0; k < NROW; ++k) load_first(pa.rowop[k], pa.ldr[k], row, in_first, r[u][k]);
            firsts[u] = in_first;
          }
          if constexpr (policy_has_val2<P>::value) {
            // (a step past the run's end reads the run's first value: a valid position)
            a2[u] = 1.f;
            if (pa.val2) a2[u] = pa.val2[it.p + (s < R.cnt ? R.start + s : 0)];
          }
        },
        [&](auto u, float a, int s) {
          if constexpr (!SEG && !PAIRS) {
            if ((P::PER_ENTRY ? firsts[u] : first) || !FIRST_ONLY) {
#pragma unroll
              for (int k = 0; k < NROW; ++k)
#pragma unroll
                for (int v = 0; v < W; ++v) rS[k][v] = r[u][k < NR ? k : 0][v];
            }
            first = false;
          }
          if constexpr (P::PER_ENTRY) {
            constexpr int k = decltype(u)::value % 4;
            share[k] = P::template partial<W, TAIL>(x[u], rS, lc);
            share_a[k] = a;
            asm volatile("" : "+v"(share[k]));  // (else the shares are formed with their sum, and their operands held until then)
            if constexpr (k == 3) park(s - 3, 4);
          } else if constexpr (PAIRS) {
            P::template apply<W>(a, sc[decltype(u)::value % 2], x[u], acc);
          } else if constexpr (policy_in_steps<P>::value) {
            constexpr int ND = P::NDOT;
            float t[2] = {}, o[2];  // (all of them, where no dot product is needed: scalars() reads them)
            if constexpr (ND > 0) {
              P::template dots<W, TAIL>(x[u], rS, lc, t);
#pragma unroll
              for (int j = 0; j < ND; ++j) t[j] = group_allreduce<LPG>(t[j]);
            }
            P::scalars(t, o);
            P::template apply<W>(a, o, x[u], acc);
          } else if constexpr (policy_has_val2<P>::value) {
            P::template edge<LPG, W, TAIL>(pa, a, a2[u], x[u], rS, acc, lc);
          } else {
            P::template edge<LPG, W, TAIL>(pa, a, x[u], rS, acc, lc);
          }
        },
        [&](int, int row) {
          first = true;
#pragma unroll
          for (int v = 0; v < W; ++v) head[v] = carried ? acc[v] : head[v];
          if (!carried) store_row(row, acc);
          carried = false;
          ended = true;
#pragma unroll
          for (int v = 0; v < W; ++v) acc[v] = 0.f;
        },
        pair);
  };
  if (it.is_seg) run(std::true_type{}); else run(std::false_type{});

  if constexpr (P::PER_ENTRY) {
    static_assert(RING % 4 == 0, "four steps at a time");
    if (R.cnt & 3) park(R.cnt & ~3, R.cnt & 3);
    wave_lds_sync();
    const int n_ent = (int)(it.p_end - it.p);
    for (int i = lane; i < n_ent; i += ISP_WAVE) {
      float* o = pa.out_entry + it.p + i;
      const float val = __int_as_float(L.ent[i].y);
      *o = P::ADD ? *o + val : val;
    }
  } else {
    if (it.is_seg) {  // one row: the groups' sums, spread over the groups (this lane stores N columns)
      constexpr int N = W / G > 0 ? W / G : 1;
      const int idx0 = group_reduce_scatter<LPG, W>(acc, lane);
      const bool on = NV == 1 ? lc.on[0] : (idx0 >= 4 ? lc.on[NV - 1] : lc.on[0]);
      if (group_owner<LPG, W>(lane) && on) {
        float t[N];
#pragma unroll
        for (int c = 0; c < N; ++c) t[c] = acc[c];
        float* row = A.partials + (int64_t)it.row * ISP_PARTIAL_TILE;
        const int c0 = idx0 >= 4 ? lc.off[NV - 1] + idx0 - 4 : lc.off[0] + idx0;
        if (finish) hf_store<N>(row, (unsigned)c0 * 4u, t);
        else store_vec<N>(row + c0, t);
      }
      // (one group adds all four quarters: with four loads in flight, one each, 200 columns and a row of 76 segments took 33.5 us, with 16 29.5,
      // in the registers that the loop holds anyway)
      if (FINISH && hf_last(A, H, 0, lane)) {
        float sum[W];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          float t[4];
          hf_sum<LPG, G == 1 ? 16 : 8>(A, H, (unsigned)lc.off[v] * 4u, lane, t);
#pragma unroll
          for (int c = 0; c < 4; ++c) sum[4 * v + c] = t[c];
        }
        if (g == 0) store_to(Y + (int64_t)it.src_row * ldy, sum);
      }
      return;
    }
    if constexpr (G > 1) {  // rows cut by a run boundary: the run in which such a row ends adds the earlier runs' sums
      const unsigned long long m_end = __ballot(ended), m_mid = __ballot(R.mid);
      const unsigned long long m_head = m_end & m_mid;
      if (m_head == 0) return;
      wave_lds_sync();  // (every entry has been read)
      float* __restrict__ tail = reinterpret_cast<float*>(L.ent);
#pragma unroll
      for (int v = 0; v < W; ++v) tail[lane * W + v] = acc[v];
      wave_lds_sync();
      if ((m_head >> lane) & 1ull) {
        int j = lane - LPG;
        for (;;) {
#pragma unroll
          for (int v = 0; v < W; ++v) head[v] += tail[j * W + v];
          if (((m_end >> j) & 1ull) || !((m_mid >> j) & 1ull)) break;  // the row began in that run
          j -= LPG;
        }
        store_row(L.dst[R.k], head);
      }
    }
  }
}

// Host side: true when a kernel over matrix columns [0, n_cols) may gather from rows of pitch ld floats
// (d columns used) with 32-bit byte offsets formed by a 24-bit multiply.
inline bool fused_offsets_fit_32(int64_t n_cols, int64_t ld, int d) {
  return n_cols < (1 << 24) && ld * 4 < (1 << 24) &&
         ((uint64_t)n_cols * (uint64_t)ld + (uint64_t)d) * 4u < ((uint64_t)1 << 32);
}

// Partial dot product of a lane's columns; vectors whose columns lie past d contribute zero, and so do the leading
// columns that a moved-back vector shares with its neighbour (three selects a vector, in the TAIL kernels only).
template <int W, bool TAIL>
__device__ inline float dotw(const float (&a)[W], const float (&b)[W], const lane_cols<W / 4, TAIL>& lc) {
  float s = 0.f;
#pragma unroll
  for (int v = 0; v < W / 4; ++v) {
    if constexpr (TAIL) {
      float p = a[4 * v + 3] * b[4 * v + 3];
      p = lc.dup[v] < 3 ? fmaf(a[4 * v + 2], b[4 * v + 2], p) : p;
      p = lc.dup[v] < 2 ? fmaf(a[4 * v + 1], b[4 * v + 1], p) : p;
      p = lc.dup[v] < 1 ? fmaf(a[4 * v], b[4 * v], p) : p;
      s += lc.on[v] ? p : 0.f;
    } else {
      const float p = fmaf(a[4 * v + 3], b[4 * v + 3], fmaf(a[4 * v + 2], b[4 * v + 2], fmaf(a[4 * v + 1], b[4 * v + 1], a[4 * v] * b[4 * v])));
      s += lc.on[v] ? p : 0.f;
    }
  }
  return s;
}

}  // namespace isp_dev
