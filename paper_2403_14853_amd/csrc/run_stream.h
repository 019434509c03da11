// Run-streaming skeleton (gfx950, wave64): the fast path of SpMM and of the min / max reductions.
//
// A wavefront owns one work item (a block of whole short rows, a block of row pieces, or one hub-row segment) whose
// nonzeros are contiguous in the CSR arrays.  The 64 lanes form G = 64 / LPG groups; a group gathers one dense row
// slice of VEC * LPG floats with one load, so one instruction serves G nonzeros.  The item's (column, value) pairs
// are staged in LDS, and every group then streams a CONTIGUOUS RUN of about n / G of them: it adds up one row after
// the other and stores a row when it has met its last entry, so
//  - every step serves G entries, wherever rows begin and end (sharing out each row's entries over the groups left
//    half of the lanes idle on rows of a few entries);
//  - a finished row costs its store, not a reduction over the groups; only the at most G rows that a run boundary
//    cuts are put together at the end, the parts in order (deterministic, no atomics);
//  - the item needs no table of steps: one ballot per 64 rows ranks the non-empty ones, one per group finds the row
//    that its run starts in.
// Empty rows own nothing in the runs; their outputs are written up front.
#pragma once
#include <limits.h>
#include <utility>
#include "group_stream.h"

namespace isp_dev {

constexpr int RN_PAD = 16;          // spare entries behind the item's last (steps of the last round may read there)
constexpr int RN_CHUNK = 2;         // entries read from LDS at a time

template <int CAP>
struct __attribute__((aligned(16))) rn_wave_lds_of {
  int2 ent[CAP + RN_PAD];          // (column, value bits); afterwards the runs' unfinished sums
  int dst[GS_MAX_ROWS + 8];        // output row of each non-empty row, in order; from the top down: the empty rows
  gs_u16 end[GS_MAX_ROWS + 8];     // where each non-empty row ends, relative to the item
};
template <int CAP>
struct rn_lds_of { rn_wave_lds_of<CAP> w[ISP_WAVES_PER_WG]; };
using rn_wave_lds = rn_wave_lds_of<GS_MAX_ENT>;
using rn_lds = rn_lds_of<GS_MAX_ENT>;

// Tables of 768 entries let a compute unit (160 KB) hold five workgroups, tables of RN_SMALL seven.  Where the items are
// that small and the dense operand fits the L2s (eight of 4 MB, shared with everything else), the additional wavefronts hide
// more of the loads' latency; where it does not fit they only spread the chip's gathers over more rows than the L2s
// keep, and a launch that does not fill five per compute unit gains nothing (per_cu: workgroups per compute unit that the launch
// must have more of; the launches' rules stand with them).  us with tables of 768 / RN_SMALL entries:
//   SpMM: 20 k columns, 400 k entries, 64 columns 14.5 / 13.7; 10 k, 1 M: 16 16.3 / 14.7, 128 33.4 / 32.2; 50 k, 1.5 M: 32 27.1 /
//   24.2, 64 35.3 / 32.6; beyond the L2s, 100 k, 1 M: 64 (26 MB) 29.4 / 30.0, 100 55.0 / 58.2;
//   SDDMM: 10 k, 1 M: 16 12.8 / 11.7, 64 18.5 / 17.1; 50 k, 1.5 M: 32 21.0 / 18.7, 64 29.9 / 27.4; beyond, 100 k, 1 M: 64 21.5 / 22.3.
constexpr int RN_SMALL = 448;
constexpr int64_t RN_FIT_BYTES = 24 << 20;
inline bool rn_small_tables(const isp_csr* A, const isp_view& v, int width, int64_t wgs, int per_cu) {
  return A->info.block_cost + v.hub_t <= RN_SMALL && v.seg_len <= RN_SMALL && v.n_cols * width * 4 <= RN_FIT_BYTES &&
         wgs * 16 > per_cu * (int64_t)A->wave_slots;  // (16 slots per compute unit)
}

// This lane's group's run, and the item's shape.
struct rn_run {
  int start, cnt;   // entries [start, start + cnt) of the item
  int k;            // index into dst of the row its first entry belongs to
  bool mid;         // the run starts inside a row: that row's sum begins in an earlier run
  int steps;        // steps in which any group has an entry (wave-uniform)
  int n_empty;      // empty rows, listed at dst[RN_EMPTY0 - i]
};
constexpr int RN_EMPTY0 = GS_MAX_ROWS + 7;

// The first 64 rows' offsets of a row block, requested before its entries so that both are on their way together.
struct rn_first_rows {
  int a, b, dst;  // of row it.row + lane: its entries [a, b) relative to the item, its output row
};
__device__ __forceinline__ rn_first_rows rn_request_rows(const item_range& it, const int64_t* __restrict__ indptr,
                                                         const int32_t* __restrict__ slot_of, int lane) {
  rn_first_rows f{0, 0, it.row + lane};
  if (!it.is_seg && lane < it.row_last - it.row) {
    f.a = (int)(indptr[it.row + lane] - it.p);
    f.b = (int)(indptr[it.row + lane + 1] - it.p);
    if (slot_of) f.dst = slot_of[it.row + lane];
  }
  return f;
}

// The groups' runs over n_ent staged entries.  slot_of: for blocks of pieces, the partial row of piece `row` (else
// NULL).  staged(o): how many of the item's first o entries are staged (all, where nothing is left out).
template <int G, class Lds, class Staged>
__device__ __forceinline__ rn_run rn_find_runs(const item_range& it, const int64_t* __restrict__ indptr,
                                               const int32_t* __restrict__ slot_of, int n_ent, const rn_first_rows& f,
                                               Staged&& staged, Lds& L, int lane) {
  const int n_rows = it.is_seg ? 0 : it.row_last - it.row;
  const int g = lane / (ISP_WAVE / G);
  const int q = n_ent / G, rest = n_ent - q * G;
  rn_run R;
  R.start = g * q + (g < rest ? g : rest);
  R.cnt = q + (g < rest ? 1 : 0);
  R.steps = q + (rest > 0 ? 1 : 0);
  R.k = 0;
  R.mid = it.is_seg;
  R.n_empty = 0;
  int live = 0;
  for (int base = 0; base < n_rows; base += ISP_WAVE) {
    const int r = base + lane;
    int a = f.a, b = f.b, dst = f.dst;
    if (base > 0) {
      a = b = 0;
      dst = it.row + r;
      if (r < n_rows) {
        a = (int)(indptr[it.row + r] - it.p);
        b = (int)(indptr[it.row + r + 1] - it.p);
        if (slot_of) dst = slot_of[it.row + r];
      }
    }
    a = staged(a);
    b = staged(b);
    const bool on = b > a;
    const unsigned long long m = __ballot(on);
    const unsigned long long below = (1ull << lane) - 1ull;
    if (on) {
      const int rank = live + __popcll(m & below);
      L.dst[rank] = dst;
      L.end[rank] = (gs_u16)b;
    }
    const unsigned long long me = __ballot(r < n_rows && !on);
    if (r < n_rows && !on) L.dst[RN_EMPTY0 - R.n_empty - __popcll(me & below)] = dst;
    R.n_empty += __popcll(me);
    const int bb = on ? b : INT_MAX;
#pragma unroll
    for (int j = 1; j < G; ++j) {  // rows that end before run j starts
      const int before = __popcll(__ballot(bb <= j * q + (j < rest ? j : rest)));
      R.k += g == j ? before : 0;
    }
    live += __popcll(m);
  }
  if (lane < 2) {  // (read ahead: a row that never ends)
    L.dst[live + lane] = 0;
    L.end[live + lane] = 0xffff;
  }
  wave_lds_sync();
  // (the last row to end before the run's first entry ends right there, or the run starts inside a row)
  if (!it.is_seg && R.cnt > 0) R.mid = R.k > 0 ? (int)L.end[R.k - 1] != R.start : R.start > 0;
  return R;
}

// Stage the item and find the groups' runs.  values may be NULL (every entry is 1).
template <int G, class Lds>
__device__ inline rn_run rn_prepare(const item_range& it, const int64_t* __restrict__ indptr,
                                    const int32_t* __restrict__ indices, const float* __restrict__ values,
                                    const int32_t* __restrict__ slot_of, Lds& L, int lane) {
  const int n_ent = (int)(it.p_end - it.p);
  const rn_first_rows f = rn_request_rows(it, indptr, slot_of, lane);
  constexpr int SB = 8;  // loads in flight per lane
  for (int base = 0; base < n_ent; base += SB * ISP_WAVE) {
    int c[SB];
    float v[SB];
#pragma unroll
    for (int u = 0; u < SB; ++u) {
      const int i = base + u * ISP_WAVE + lane;
      c[u] = 0;
      v[u] = 1.f;
      if (i < n_ent) {
        c[u] = __builtin_nontemporal_load(indices + it.p + i);
        if (values) v[u] = __builtin_nontemporal_load(values + it.p + i);
      }
    }
#pragma unroll
    for (int u = 0; u < SB; ++u) {
      const int i = base + u * ISP_WAVE + lane;
      if (i < n_ent) L.ent[i] = make_int2(c[u], __float_as_int(v[u]));
    }
  }
  if (lane < RN_PAD) L.ent[n_ent + lane] = make_int2(0, 0);
  return rn_find_runs<G>(it, indptr, slot_of, n_ent, f, [](int o) { return o; }, L, lane);
}

// f(0) ... f(N - 1) with the index as a compile-time constant (ring slots live in registers).
template <class F, int... U>
__device__ __forceinline__ void rn_for_each(F&& f, std::integer_sequence<int, U...>) { (f(std::integral_constant<int, U>{}), ...); }
template <int N, class F>
__device__ __forceinline__ void rn_for(F&& f) { rn_for_each(f, std::make_integer_sequence<int, N>{}); }

// A cursor over a run's rows: the row of the current step, the step that ends it, and the row after it (read one row
// ahead, so that nothing waits for the list).
struct rn_cursor {
  int k, row, row_next, end, end_next;
  template <class Lds>
  __device__ __forceinline__ rn_cursor(const Lds& L, const rn_run& R)
      : k(R.k), row(L.dst[R.k]), row_next(L.dst[R.k + 1]), end((int)L.end[R.k] - R.start - 1), end_next(L.end[R.k + 1]) {}
  template <class Lds>
  __device__ __forceinline__ void advance(const Lds& L, const rn_run& R) {
    ++k;
    row = row_next;
    end = end_next - R.start - 1;
    row_next = L.dst[k + 1];
    end_next = L.end[k + 1];
  }
};

// Stream the runs.  load(u, col, s, row, first): request what ring slot u needs of entry s of the run, which lies in row `row`
// (ROWS only: else 0);  add(u, a, s): take slot u (a compile-time constant) into the running result, a the entry's value;  end_row(k, row): the
// k-th non-empty row is complete in this lane's group, its output row is `row` (ENDS only; called by the lanes it
// concerns only).  RING steps are in flight per lane.
// A round of RING steps is consumed while the next one is requested, slot by slot, into the same registers; the
// entries are read from LDS CHUNK steps before they are needed.  A row's end is the step number at which it
// ends, kept per lane: one comparison a step.
// PAIRS: slots are taken and requested again two at a time; pair(u) comes before add(u) and add(u + 1), of which the second is
// left out (and what slot u + 1 holds means nothing) where a run ends with slot u.
struct rn_no_pairs {
  template <class U>
  __device__ __forceinline__ void operator()(U) const {}
};
template <int RING, bool ENDS, bool ROWS, int CHUNK = RN_CHUNK, bool PAIRS = false, class Lds, class Load, class Add, class End,
          class Pair = rn_no_pairs>
__device__ __forceinline__ void rn_stream(const Lds& L, const rn_run& R, Load&& load, Add&& add, End&& end_row, Pair&& pair = Pair()) {
  static_assert(RING % (2 * CHUNK) == 0 && 2 * CHUNK <= RN_PAD, "fetches alternate between two buffers");
  const int2* __restrict__ ep = L.ent + R.start;
  constexpr int C = CHUNK;
  float a[RING];
  int2 e[2][C];  // entries to request next, and the ones after them
  rn_cursor out(L, R), in(L, R);
  bool in_first = true;  // (ROWS) the step to request next is its row's first in this run
  auto fetch = [&](int2 (&o)[C], int s0) {
#pragma unroll
    for (int u = 0; u < C; ++u) o[u] = ep[s0 + u];
  };
  auto request = [&](int u, const int2& n, int s) {
    load(u, n.x, s, ROWS ? in.row : 0, in_first);
    a[u] = __int_as_float(n.y);
    if constexpr (ROWS) {
      in_first = in.end == s;
      if (in_first) in.advance(L, R);
    }
  };
  auto take = [&](auto u, int s0) {
    add(u, a[u], s0 + u);
    if constexpr (ENDS)
      if (out.end == s0 + u) {
        end_row(out.k, out.row);
        out.advance(L, R);
      }
  };
  auto take_pair = [&](auto u, int s0, bool both) {  // slots u, u + 1
    pair(u);
    take(u, s0);
    if (both) take(std::integral_constant<int, decltype(u)::value + 1>{}, s0);
  };
  static_assert(!PAIRS || (RING % 2 == 0 && CHUNK == 2), "a pair's entries are read together");
  // Requests behind a condition make the compiler wait for everything in flight, so the steady state has none.  The
  // steps left over after the last whole round do ask whether there is a step.
  const int rounds = R.steps / RING, rest = R.steps - rounds * RING;  // wave-uniform
  if (rounds + rest == 0) return;
  fetch(e[0], 0);
  int s0 = 0;  // steps consumed so far
  if (rounds > 0) {
    rn_for<RING>([&](auto u) {
      if constexpr (u % C == 0) fetch(e[(u / C + 1) & 1], u + C);
      request(u, e[(u / C) & 1][u % C], u);
    });
    for (int r = 1; r < rounds; ++r, s0 += RING) {
      rn_for<RING>([&](auto u) {
        if constexpr (u % C == 0) fetch(e[(u / C + 1) & 1], s0 + RING + u + C);
        if constexpr (!PAIRS) {
          take(u, s0);
          request(u, e[(u / C) & 1][u % C], s0 + RING + u);
        } else if constexpr (u % 2 == 0) {
          take_pair(u, s0, true);
          request(u, e[(u / C) & 1][0], s0 + RING + u);
          request(u + 1, e[(u / C) & 1][1], s0 + RING + u + 1);
        }
      });
    }
    if (rest > 0) {
      rn_for<RING>([&](auto u) {
        if constexpr (u % C == 0) fetch(e[(u / C + 1) & 1], s0 + RING + u + C);
        if constexpr (!PAIRS) take(u, s0);
        else if constexpr (u % 2 == 0) take_pair(u, s0, true);
        if (u < rest) request(u, e[(u / C) & 1][u % C], s0 + RING + u);
      });
      s0 += RING;
    }
  } else {
    rn_for<RING>([&](auto u) {
      if constexpr (u % C == 0) fetch(e[(u / C + 1) & 1], u + C);
      if (u < rest) request(u, e[(u / C) & 1][u % C], u);
    });
  }
  const int left = R.cnt - s0;  // of this lane's run
  rn_for<RING>([&](auto u) {
    if constexpr (!PAIRS) {
      if (u < left) take(u, s0);
    } else if constexpr (u % 2 == 0) {
      if (u < left) take_pair(u, s0, u + 1 < left);
    }
  });
}

}  // namespace isp_dev
