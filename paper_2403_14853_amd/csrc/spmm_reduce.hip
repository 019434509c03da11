// Sparse-dense product with the other reductions the paper's matmul offers (Section 3.4, 3.5):
// mean, min, max - and their backward through the cached transpose.  The sum reduction has the tuned
// kernels and mean reuses them (rows divided by their length); min / max have run-streaming kernels of the same
// design, forward and backward, from 4 columns up at any alignment where gather offsets fit 32 bits.  The rest
// runs on the generic row-streaming skeleton (one nonzero per wave iteration, any width and alignment).
//   mean : Y[i] = (sum_p a_p x_j) / len_i
//   min / max : Y[i,k] = min / max_p a_p x_jk (product and comparison in fp32), arg[i,k] = position p of
//               the first entry attaining it; empty row -> 0 and -1
//   backward mean    : dX[j] = sum_{p in column j} (a_p / len_row(p)) dY[row(p)]
//   backward min/max : dX[j,k] = sum_{p in column j, arg[row(p),k] == p} a_p dY[row(p),k]
// Both backward forms are row passes over the cached transpose (whose perm gives p), so no
// floating-point atomics are needed and results are deterministic.
#include "row_stream.h"
#include "hub_finish.h"
#include "lane_rule.h"
#include "run_stream.h"

namespace {
using namespace isp_dev;

constexpr int R_MEAN = 1, R_MIN = 2, R_MAX = 3;
constexpr int ARG_OFF = ISP_PARTIAL_TILE / 2;  // hub partial rows: values in [0,128), arg bits in [128,256)

// ---- forward -----------------------------------------------------------------------------------
template <int VEC_, int MODE, bool HAS_VAL_>
struct reduce_fwd_policy {
  static constexpr int VEC = VEC_, T = 1, NG = 1, U = 8;
  static constexpr bool HAS_VAL = HAS_VAL_, ACCUMULATE = false, NEEDS_PERM = false, HAS_FINISH = true;
  struct args { const float* src[1]; int64_t ld[1]; int32_t* arg; int d; const int32_t* perm; };
  struct row_state { int where[VEC]; };
  __device__ static inline void row_begin(const args&, row_state& rs, int, const int (&)[1], const bool (&)[1]) {
#pragma unroll
    for (int v = 0; v < VEC; ++v) rs.where[v] = -1;
  }
  __device__ static inline void edge(const args&, row_state& rs, float a, const float (&x)[1][1][VEC],
                                     float (&acc)[1][VEC], const bool (&)[1], const edge_info& ei) {
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
      if (MODE == R_MEAN) {
        acc[0][v] = fmaf(a, x[0][0][v], acc[0][v]);
      } else {
        const float t = __fmul_rn(a, x[0][0][v]);  // one rounded fp32 multiply, never fused
        const bool take = rs.where[v] < 0 || (MODE == R_MIN ? t < acc[0][v] : t > acc[0][v]);
        acc[0][v] = take ? t : acc[0][v];
        rs.where[v] = take ? (int)ei.pos : rs.where[v];
      }
    }
  }
  __device__ static inline void finish(const args& pa, row_state& rs, float (&acc)[1][VEC], int out_row, bool is_seg,
                                       int64_t row_len, float* side, const int (&col)[1], const bool (&on)[1],
                                       int k0) {
    if (MODE == R_MEAN) {
      if (!is_seg) {  // segments hold plain partial sums; the fix-up divides
        const float inv = row_len > 0 ? 1.f / (float)row_len : 0.f;
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[0][v] *= inv;
      }
    } else if (on[0]) {
      // an empty row never saw row_begin: its position is -1 by definition
      const bool empty = !is_seg && row_len == 0;
#pragma unroll
      for (int v = 0; v < VEC; ++v) {
        const int w = empty ? -1 : rs.where[v];
        if (is_seg) side[ARG_OFF + col[0] - k0 + v] = __int_as_float(w);
        else pa.arg[(int64_t)out_row * pa.d + col[0] + v] = w;
      }
    }
#pragma unroll
    for (int v = 0; v < VEC; ++v) rs.where[v] = -1;
  }
};

template <int VEC, int MODE, bool HAS_VAL>
__global__ void __launch_bounds__(ISP_WG) k_reduce_fwd(isp_view A, const int64_t* __restrict__ indptr,
                                                       const int32_t* __restrict__ indices,
                                                       const float* __restrict__ values, const float* __restrict__ X,
                                                       int64_t ldx, int d, int k0, float* __restrict__ Y, int64_t ldy,
                                                       int32_t* __restrict__ arg) {
  using P = reduce_fwd_policy<VEC, MODE, HAS_VAL>;
  typename P::args pa;
  pa.src[0] = X; pa.ld[0] = ldx; pa.arg = arg; pa.d = d; pa.perm = nullptr;
  stream_item<P>(A, indptr, indices, values, pa, d, k0, Y, ldy);
}

// ---- run-streaming forward of min / max ------------------------------------------------------------------
// The SpMM kernel's items and runs (run_stream.h) with the sum replaced by a running (value, position) pair per
// column.  A run meets its entries in ascending position, so "replace only if strictly better" keeps the first
// entry of a row that attains the extremum; the parts of a row that a run boundary cuts are put together with the
// earlier part kept unless the later one is better.  Hub segments leave (value, position) halves in their
// partial rows exactly as the generic kernel does, and the same fix-up combines them in segment order.
// Needs 4 columns or more and 32-bit gather offsets; a launch covers at most 128 columns (the partial rows).
// Bound by the vector ALU on short rows (a comparison and two selects per column and entry, and the row ends): with
// every row's entries shared out over the groups and a reduction of pairs at every row end 2.4 M entries took
// 216 us at 16 columns and 159 at 64, now 34 and 67.
template <int MODE>
__device__ inline bool mm_better(float t, float best) { return MODE == R_MIN ? t < best : t > best; }

constexpr int MINMAX_RING = 4;

// FINISH: hub rows are put together here (hub_finish.h), with the results of the fix-up's fold in segment order, bit for bit.
template <int LPG, int MODE, bool FINISH>
__global__ void __launch_bounds__(ISP_WG) k_minmax_grouped(isp_view A, const int64_t* __restrict__ indptr,
                                                           const int32_t* __restrict__ indices,
                                                           const float* __restrict__ values,
                                                           const float* __restrict__ X, int64_t ldx, int d, int k_base,
                                                           float* __restrict__ Y, int64_t ldy,
                                                           int32_t* __restrict__ arg) {
  constexpr int G = ISP_WAVE / LPG;
  __shared__ rn_lds lds;
  const int lane = threadIdx.x & (ISP_WAVE - 1);
  const int w = threadIdx.x >> 6;
  const int item = __builtin_amdgcn_readfirstlane((int)blockIdx.x * ISP_WAVES_PER_WG + w);
  if (item >= A.n_blocks + A.n_seg) return;
  const item_range it = locate_item(A, indptr, item);
  if (it.skip) return;
  rn_wave_lds& L = lds.w[w];
  const bool finish = FINISH && it.is_seg;
  hub_ref H{0, 0, 0};
  if (finish) H.h = A.seg_hub[it.row];
  const rn_run R = rn_prepare<G>(it, indptr, indices, values, nullptr, L, lane);
  if (finish) {
    H.s0 = A.hub_seg_ptr[H.h];
    H.s1 = A.hub_seg_ptr[H.h + 1];
  }

  const int g = lane / LPG, q = lane % LPG;
  // (lanes past d work on the last columns again and store what the columns' own lane stores)
  const int col = k_base + tail_col<4>(q * 4, d - k_base);
  const unsigned lane_byte = (unsigned)col * 4u;
  const unsigned pitch_byte = (unsigned)ldx * 4u;
  const int p0 = (int)it.p;  // position of the item's first entry (nnz < 2^31)

  float best[4], head[4], x[MINMAX_RING][4];
  int where[4], head_where[4];  // entry's number in the run until a row ends, then its position
#pragma unroll
  for (int v = 0; v < 4; ++v) { best[v] = head[v] = 0.f; where[v] = head_where[v] = -1; }
  auto store_row = [&](int row, const float (&b)[4], const int (&wh)[4]) {
    float wb[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) wb[v] = __int_as_float(wh[v]);
    if (it.is_seg) {
      float* pr = A.partials + (int64_t)row * ISP_PARTIAL_TILE + (col - k_base);
      store_vec<4>(pr, b);
      store_vec<4>(pr + ARG_OFF, wb);
    } else {
      store_vec<4>(Y + (int64_t)row * ldy + col, b);
      store_vec<4>(reinterpret_cast<float*>(arg) + (int64_t)row * d + col, wb);
    }
  };
  for (int i = g; i < R.n_empty; i += G) store_row(L.dst[RN_EMPTY0 - i], best, where);  // value 0, position -1

  bool carried = R.mid;  // the next row to end began in an earlier run
  bool ended = false;    // a row has ended in this run
  bool fresh = true;     // no entry of the current row has been met in this run
  const int pos0 = p0 + R.start;
  rn_stream<MINMAX_RING, true, false>(
      L, R,
      [&](int u, int c, int, int, bool) {
        const unsigned off = __umul24((unsigned)c, pitch_byte) + lane_byte;
        load_vec<4>(reinterpret_cast<const float*>(reinterpret_cast<const char*>(X) + off), x[u]);
      },
      [&](int u, float a, int s) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float t = __fmul_rn(a, x[u][v]);  // one rounded fp32 multiply, never fused
          const bool take = fresh || mm_better<MODE>(t, best[v]);
          best[v] = take ? t : best[v];
          where[v] = take ? s : where[v];
        }
        fresh = false;
      },
      [&](int, int row) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          where[v] += pos0;
          head[v] = carried ? best[v] : head[v];
          head_where[v] = carried ? where[v] : head_where[v];
        }
        if (!carried) store_row(row, best, where);
        carried = false;
        ended = true;
        fresh = true;
      });
#pragma unroll
  for (int v = 0; v < 4; ++v) where[v] = fresh ? -1 : where[v] + pos0;

  if (it.is_seg) {  // one row: the groups' pairs, ties going to the smaller position
#pragma unroll
    for (int o = LPG; o < ISP_WAVE; o <<= 1) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float ob = __shfl_xor(best[v], o);
        const int ow = __shfl_xor(where[v], o);
        const bool take = ow >= 0 && (where[v] < 0 || mm_better<MODE>(ob, best[v]) || (ob == best[v] && ow < where[v]));
        best[v] = take ? ob : best[v];
        where[v] = take ? ow : where[v];
      }
    }
    if constexpr (FINISH) {
      float* row = A.partials + (int64_t)it.row * ISP_PARTIAL_TILE;
      const unsigned byte = (unsigned)(col - k_base) * 4u;
      if (g == 0) {
        float wb[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) wb[v] = __int_as_float(where[v]);
        hf_store<4>(row, byte, best);
        hf_store<4>(row, byte + ARG_OFF * 4u, wb);
      }
      if (!hf_last(A, H, 0, lane)) return;
      // Each group folds a contiguous part of the segments.  A NaN decides only as the row's first segment (nothing is better than it,
      // and it is better than nothing): the later parts pass over theirs.
      const int n = H.s1 - H.s0, part = (n + G - 1) / G, first = g * part, end = first + part < n ? first + part : n;
      float* base = A.partials + (int64_t)H.s0 * ISP_PARTIAL_TILE;
      constexpr int U = 8;  // partial rows in flight
#pragma unroll
      for (int v = 0; v < 4; ++v) where[v] = -1;
      for (int i = 0; i < part; i += U) {
        float t[U][4], wb[U][4];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int s = first + i + u < n ? first + i + u : n - 1;
          const unsigned at = (unsigned)s * (unsigned)(ISP_PARTIAL_TILE * 4) + byte;
          hf_load(base, at, t[u]);
          hf_load(base, at + ARG_OFF * 4u, wb[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const bool start = where[v] < 0 && (g == 0 || t[u][v] == t[u][v]);
            const bool take = first + i + u < end && i + u < part && (start || (where[v] >= 0 && mm_better<MODE>(t[u][v], best[v])));
            best[v] = take ? t[u][v] : best[v];
            where[v] = take ? __float_as_int(wb[u][v]) : where[v];
          }
      }
#pragma unroll
      for (int o = LPG; o < ISP_WAVE; o <<= 1) {  // neighbouring parts, the earlier one kept unless the later one is better
        const bool later = (lane & o) != 0;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float ob = __shfl_xor(best[v], o);
          const int ow = __shfl_xor(where[v], o);
          const float eb = later ? ob : best[v], lb = later ? best[v] : ob;
          const int ew = later ? ow : where[v], lw = later ? where[v] : ow;
          const bool take = lw >= 0 && (ew < 0 || mm_better<MODE>(lb, eb));
          best[v] = take ? lb : eb;
          where[v] = take ? lw : ew;
        }
      }
      if (g == 0) {
        float wb[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) wb[v] = __int_as_float(where[v]);
        store_vec<4>(Y + (int64_t)it.src_row * ldy + col, best);
        store_vec<4>(reinterpret_cast<float*>(arg) + (int64_t)it.src_row * d + col, wb);
      }
    } else if (g == 0) {
      store_row(it.row, best, where);
    }
    return;
  }
  if constexpr (G > 1) {  // rows cut by a run boundary (as in k_spmm_grouped)
    const unsigned long long m_end = __ballot(ended), m_mid = __ballot(R.mid);
    const unsigned long long m_head = m_end & m_mid;
    if (m_head == 0) return;
    wave_lds_sync();  // (every entry has been read)
    float* __restrict__ tail = reinterpret_cast<float*>(L.ent);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      tail[lane * 8 + v] = best[v];
      tail[lane * 8 + 4 + v] = __int_as_float(where[v]);
    }
    wave_lds_sync();
    if ((m_head >> lane) & 1ull) {
      int j = lane - LPG;
      for (;;) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float tb = tail[j * 8 + v];
          const int tw = __float_as_int(tail[j * 8 + 4 + v]);
          const bool later = mm_better<MODE>(head[v], tb);
          head[v] = later ? head[v] : tb;
          head_where[v] = later ? head_where[v] : tw;
        }
        if (((m_end >> j) & 1ull) || !((m_mid >> j) & 1ull)) break;  // the row began in that run
        j -= LPG;
      }
      store_row(L.dst[R.k], head, head_where);
    }
  }
}

// One wave per hub row: combine the segments' partial results in segment order.
template <int VEC, int MODE>
__global__ void __launch_bounds__(ISP_WG) k_reduce_fixup(isp_view A, int d, int k0, float* __restrict__ Y, int64_t ldy,
                                                         int32_t* __restrict__ arg) {
  const int lane = threadIdx.x & (ISP_WAVE - 1);
  const int h = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * ISP_WAVES_PER_WG + (threadIdx.x >> 6)));
  if (h >= A.n_hub) return;
  const int s0 = A.hub_seg_ptr[h], s1 = A.hub_seg_ptr[h + 1];
  const int row = A.hub_rows[h];
  if (k0 + lane * VEC >= d) return;
  const int rel = tail_col<VEC>(lane * VEC, d - k0);
  float best[VEC];
  int where[VEC];
#pragma unroll
  for (int v = 0; v < VEC; ++v) { best[v] = 0.f; where[v] = -1; }
  auto combine = [&](const float (&t)[VEC], const float (&wbits)[VEC]) {
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
      if (MODE == R_MEAN) {
        best[v] += t[v];
      } else {
        const bool take = where[v] < 0 || (MODE == R_MIN ? t[v] < best[v] : t[v] > best[v]);
        best[v] = take ? t[v] : best[v];
        where[v] = take ? __float_as_int(wbits[v]) : where[v];
      }
    }
  };
  int s = s0;
  for (; s + 8 <= s1; s += 8) {  // eight segments' partial rows in flight, combined in segment order
    float t[8][VEC], wb[8][VEC];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const float* pr = A.partials + (int64_t)(s + u) * ISP_PARTIAL_TILE + rel;
      load_vec<VEC>(pr, t[u]);
      if (MODE != R_MEAN) load_vec<VEC>(pr + ARG_OFF, wb[u]);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) combine(t[u], wb[u]);
  }
  for (; s < s1; ++s) {
    const float* pr = A.partials + (int64_t)s * ISP_PARTIAL_TILE + rel;
    float t[VEC], wb[VEC];
    load_vec<VEC>(pr, t);
    if (MODE != R_MEAN) load_vec<VEC>(pr + ARG_OFF, wb);
    combine(t, wb);
  }
  if (MODE == R_MEAN) {
    const int64_t len = A.indptr[row + 1] - A.indptr[row];
    const float inv = len > 0 ? 1.f / (float)len : 0.f;
#pragma unroll
    for (int v = 0; v < VEC; ++v) best[v] *= inv;
  }
#pragma unroll
  for (int v = 0; v < VEC; ++v) {
    Y[(int64_t)row * ldy + k0 + rel + v] = best[v];
    if (MODE != R_MEAN) arg[(int64_t)row * d + k0 + rel + v] = where[v];
  }
}

// ---- backward (row passes over the cached transpose) ---------------------------------------------
// mean: entry (j <- i) contributes (a / len_A(i)) dY[i]; len_A from the source matrix's row offsets.
template <int VEC_, bool HAS_VAL_>
struct mean_bwd_policy {
  static constexpr int VEC = VEC_, T = 1, NG = 1, U = 8;
  static constexpr bool HAS_VAL = HAS_VAL_, ACCUMULATE = false, NEEDS_PERM = false, HAS_FINISH = false;
  struct args { const float* src[1]; int64_t ld[1]; const int64_t* src_indptr; const int32_t* perm; };
  struct row_state {};
  __device__ static inline void row_begin(const args&, row_state&, int, const int (&)[1], const bool (&)[1]) {}
  __device__ static inline void edge(const args& pa, row_state&, float a, const float (&x)[1][1][VEC],
                                     float (&acc)[1][VEC], const bool (&)[1], const edge_info& ei) {
    const int64_t len = pa.src_indptr[ei.col + 1] - pa.src_indptr[ei.col];
    const float w = a / (float)len;  // len >= 1: the entry itself lies in that row
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[0][v] = fmaf(w, x[0][0][v], acc[0][v]);
  }
};

// min / max: gathers dY[i] and arg[i] (as bit patterns); the entry contributes where arg equals its
// position p = perm[q] in the source matrix.  An entry that no column of its row selected (live[q] == 0,
// marked from arg before the pass) is passed over without gathering anything: in a row of many entries at
// most d of them are selected.
template <int VEC_, bool HAS_VAL_>
struct select_bwd_policy {
  static constexpr int VEC = VEC_, T = 1, NG = 2, U = 4;
  static constexpr bool HAS_VAL = HAS_VAL_, ACCUMULATE = false, NEEDS_PERM = true, HAS_FINISH = false, HAS_SKIP = true;
  struct args { const float* src[2]; int64_t ld[2]; const int32_t* perm; const uint8_t* live; };
  struct row_state {};
  __device__ static inline void row_begin(const args&, row_state&, int, const int (&)[1], const bool (&)[1]) {}
  __device__ static inline void edge(const args&, row_state&, float a, const float (&x)[2][1][VEC],
                                     float (&acc)[1][VEC], const bool (&)[1], const edge_info& ei) {
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
      const bool mine = __float_as_int(x[1][0][v]) == ei.perm;
      acc[0][v] = mine ? fmaf(a, x[0][0][v], acc[0][v]) : acc[0][v];
    }
  }
};

template <class P>
__global__ void __launch_bounds__(ISP_WG) k_reduce_bwd(isp_view At, const int64_t* __restrict__ indptr,
                                                       const int32_t* __restrict__ indices,
                                                       const float* __restrict__ values, typename P::args pa, int d,
                                                       int k0, float* __restrict__ dX, int64_t lddx) {
  stream_item<P>(At, indptr, indices, values, pa, d, k0, dX, lddx);
}

// The same pass on contiguous runs (run_stream.h), for widths from 4 columns and 32-bit offsets.  Only the live
// entries of an item are staged (packed with ballots; a row's end is the number of live entries before it), so the
// loop sees a short matrix without dead entries, G of them per step, and a row without live entries is an empty one.
// Of dY and arg a live entry gathers only the eighths of the slice that the marks name: a row of 50 entries and 100
// columns selects two or three columns per entry.  Bound by these gathers on large graphs.  The whole backward, us,
// against one entry per wavefront and iteration -> whole rows of live entries -> their marked eighths: 40 M entries, 100
// columns 2335 -> 1951 -> 1371; 115 M, 64 columns 1665 -> 1679 -> 1250; 2.4 M, 16 / 100 columns 142 -> 56 -> 51 /
// 255 -> 179 -> 141.
template <bool HAS_VAL>
struct sel_wave_lds {
  rn_wave_lds rn;                     // ent: (column | marks of the lanes that selected the entry << 24, source position)
  float val[HAS_VAL ? GS_MAX_ENT + RN_PAD : 1];  // value of each staged entry
  unsigned long long mask[GS_MAX_ENT / ISP_WAVE + 1];  // live entries of each 64 of the item ...
  int before[GS_MAX_ENT / ISP_WAVE + 1];               // ... and how many live ones precede them
};

constexpr int SELECT_RING = 4;
constexpr int SELECT_WAVES = 2;  // per workgroup: the LDS then holds 16 wavefronts per CU (14 with values), not 12

// The mark of a lane's columns in an entry's byte: eight parts of a row's slice, 64 bytes each with 32 lanes (memory
// fetches no less).
template <int LPG>
__device__ __forceinline__ int lane_part(int q) { return q * 8 / LPG; }

// marks[inv_perm[p]] = the eighths of the row slice whose columns of arg name p, for the columns from k_base; marks was zeroed
// before.  A wavefront takes a row block of A, whose rows name only the block's own entries, and gathers their marks in
// LDS, a byte per eighth (bits set by LDS atomics queue up: in a row of 14 entries 100 columns meet on 14 words, 71 us
// against 23 on 2.4 M entries); or one hub row, which has at most as many selected entries as columns and marks them whole.  (What a
// caller's array may hold besides - the -1 of empty rows, positions elsewhere - is ignored; a mark too many costs a look
// at arg.)  Bound by the scattered bytes: 40 M entries, 100 columns 227 us (363 with
// a lookup per row and column).
constexpr int MARK_ROWS = 4;  // rows per lane group in flight (8: 1 % slower, blocks of few rows load in vain)

template <int LPG>
__global__ void __launch_bounds__(ISP_WG) k_mark_lanes(isp_view A, const int64_t* __restrict__ indptr,
                                                       const int32_t* __restrict__ arg, int d, int k_base,
                                                       const int32_t* __restrict__ inv_perm, uint8_t* __restrict__ marks) {
  constexpr int G = ISP_WAVE / LPG, U = MARK_ROWS;
  __shared__ uint2 lds[ISP_WAVES_PER_WG][GS_MAX_ENT];  // a byte per entry and part
  const int lane = threadIdx.x & (ISP_WAVE - 1);
  const int w = threadIdx.x >> 6;
  const int item = __builtin_amdgcn_readfirstlane((int)blockIdx.x * ISP_WAVES_PER_WG + w);
  if (item >= A.n_blocks) {
    if (item >= A.n_blocks + A.n_hub) return;
    const int row = A.hub_rows[item - A.n_blocks];
    const int64_t p0 = indptr[row], p1 = indptr[row + 1];
    const int k_end = d < k_base + 4 * LPG ? d : k_base + 4 * LPG;
    for (int k = k_base + lane; k < k_end; k += ISP_WAVE) {
      const int p = arg[(int64_t)row * d + k];
      if (p >= p0 && p < p1) marks[inv_perm[p]] = 0xff;
    }
    return;
  }
  const item_range it = locate_item(A, indptr, item);
  if (it.skip) return;
  uint2* __restrict__ m = lds[w];
  const unsigned n = (unsigned)(it.p_end - it.p), p0 = (unsigned)it.p;
  for (unsigned i = lane; i < n; i += ISP_WAVE) m[i] = make_uint2(0u, 0u);
  wave_lds_sync();
  const int g = lane / LPG, q = lane % LPG;
  const int col = k_base + tail_col<4>(q * 4, d - k_base);
  uint8_t* __restrict__ mine = reinterpret_cast<uint8_t*>(m) + lane_part<LPG>(q);
  for (int r = it.row + g; r < it.row_last; r += G * U) {
    int where[U][4];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int row = r + u * G < it.row_last ? r + u * G : it.row_last - 1;
      float t[4];
      load_vec<4>(reinterpret_cast<const float*>(arg) + (int64_t)row * d + col, t);
#pragma unroll
      for (int v = 0; v < 4; ++v) where[u][v] = __float_as_int(t[v]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const unsigned i = (unsigned)where[u][v] - p0;
        if (i < n && r + u * G < it.row_last) mine[i * 8u] = 1;
      }
  }
  wave_lds_sync();
  for (unsigned i = lane; i < n; i += ISP_WAVE) {
    const uint2 b = m[i];
    // (the low bits of four bytes: the product's bits 24 to 27)
    const unsigned parts = (b.x * 0x01020408u >> 24 & 15u) | (b.y * 0x01020408u >> 20 & 240u);
    if (parts) marks[inv_perm[it.p + i]] = (uint8_t)parts;
  }
}

// FINISH: hub rows are put together here (hub_finish.h; us of the whole backward with the fix-up / without: 2 k rows, 20 k entries:
// 16 columns 13.7 / 11.0, 100 18.5 / 15.7; 10 k, 300 k: 16 18.1 / 15.7, 128 28.6 / 25.9; 100 k, 1 M: 32 35.4 / 32.9, 128 87.6 / 85.4).
template <int LPG, bool HAS_VAL, bool FINISH>
__global__ void __launch_bounds__(SELECT_WAVES * ISP_WAVE) k_select_grouped(isp_view At, const int64_t* __restrict__ indptr,
                                                           const int32_t* __restrict__ indices,
                                                           const float* __restrict__ values,
                                                           const int32_t* __restrict__ perm,
                                                           const uint8_t* __restrict__ marks,
                                                           const float* __restrict__ dY, int64_t lddy,
                                                           const int32_t* __restrict__ arg, int d, int k_base,
                                                           float* __restrict__ dX, int64_t lddx) {
  constexpr int G = ISP_WAVE / LPG;
  __shared__ sel_wave_lds<HAS_VAL> lds[SELECT_WAVES];
  const int lane = threadIdx.x & (ISP_WAVE - 1);
  const int w = threadIdx.x >> 6;
  const int item = __builtin_amdgcn_readfirstlane((int)blockIdx.x * SELECT_WAVES + w);
  if (item >= At.n_blocks + At.n_seg) return;
  const item_range it = locate_item(At, indptr, item);
  if (it.skip) return;
  sel_wave_lds<HAS_VAL>& S = lds[w];
  rn_wave_lds& L = S.rn;
  const int n_all = (int)(it.p_end - it.p);
  const bool finish = FINISH && it.is_seg;
  hub_ref H{0, 0, 0};
  if (finish) H.h = At.seg_hub[it.row];
  const rn_first_rows f = rn_request_rows(it, indptr, nullptr, lane);
  // stage the live entries: all the marks first, then what the live ones need
  constexpr int SB = GS_MAX_ENT / ISP_WAVE;
  unsigned char on[SB];
#pragma unroll
  for (int u = 0; u < SB; ++u) {
    const int i = u * ISP_WAVE + lane;
    on[u] = 0;
    if (u * ISP_WAVE < n_all && i < n_all) on[u] = marks[it.p + i];
  }
  int n_ent = 0;
#pragma unroll
  for (int u = 0; u < SB; ++u) {
    const unsigned long long m = __ballot(on[u] != 0);
    if (lane == 0) { S.mask[u] = m; S.before[u] = n_ent; }
    if (on[u] != 0) {
      const int64_t p = it.p + u * ISP_WAVE + lane;
      const int o = n_ent + __popcll(m & ((1ull << lane) - 1ull));
      L.ent[o] = make_int2((int)((unsigned)indices[p] | (unsigned)on[u] << 24), perm[p]);
      if (HAS_VAL) S.val[o] = values[p];
    }
    n_ent += __popcll(m);
  }
  if (finish) {
    H.s0 = At.hub_seg_ptr[H.h];
    H.s1 = At.hub_seg_ptr[H.h + 1];
  }
  if (lane == 0) { S.mask[SB] = 0; S.before[SB] = n_ent; }
  if (lane < RN_PAD) L.ent[n_ent + lane] = make_int2(0, 0);
  wave_lds_sync();
  const rn_run R = rn_find_runs<G>(it, indptr, nullptr, n_ent, f, [&](int o) {
    return S.before[o >> 6] + __popcll(S.mask[o >> 6] & ((1ull << (o & 63)) - 1ull));
  }, L, lane);

  const int g = lane / LPG, q = lane % LPG;
  const int col = k_base + tail_col<4>(q * 4, d - k_base);
  const unsigned mine = 1u << (24 + lane_part<LPG>(q));
  float* __restrict__ out = it.is_seg ? At.partials + (col - k_base) : dX + col;
  const int64_t ldo = it.is_seg ? (int64_t)ISP_PARTIAL_TILE : lddx;
  float acc[4] = {0.f, 0.f, 0.f, 0.f}, head[4] = {0.f, 0.f, 0.f, 0.f};
  for (int i = g; i < R.n_empty; i += G) store_vec<4>(out + (int64_t)L.dst[RN_EMPTY0 - i] * ldo, acc);

  float x[SELECT_RING][4], wh[SELECT_RING][4], val[SELECT_RING];
  unsigned key[SELECT_RING];
  bool carried = R.mid, ended = false;  // (as in k_spmm_grouped)
  rn_stream<SELECT_RING, true, false>(
      L, R,
      [&](int u, int c, int s, int, bool) {
        // (a lane without a mark reads the first row's first columns, which stay in the L1: no branch around the loads)
        key[u] = (unsigned)c;
        const bool on = (key[u] & mine) != 0;
        const unsigned cb = (unsigned)col * 4u;
        const unsigned oy = on ? __umul24(key[u], (unsigned)lddy * 4u) + cb : 0u;  // (the product takes the low 24 bits)
        const unsigned oa = on ? __umul24(key[u], (unsigned)d * 4u) + cb : 0u;
        load_vec<4>(reinterpret_cast<const float*>(reinterpret_cast<const char*>(dY) + oy), x[u]);
        load_vec<4>(reinterpret_cast<const float*>(reinterpret_cast<const char*>(arg) + oa), wh[u]);
        if (HAS_VAL) val[u] = S.val[R.start + s];
      },
      [&](int u, float a, int) {  // (a: the entry's source position, as bits)
        const bool on = (key[u] & mine) != 0;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const bool take = on && __float_as_int(wh[u][v]) == __float_as_int(a);
          const float sum = HAS_VAL ? fmaf(val[u], x[u][v], acc[v]) : acc[v] + x[u][v];
          acc[v] = take ? sum : acc[v];
        }
      },
      [&](int, int row) {
#pragma unroll
        for (int v = 0; v < 4; ++v) head[v] = carried ? acc[v] : head[v];
        if (!carried) store_vec<4>(out + (int64_t)row * ldo, acc);
        carried = false;
        ended = true;
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[v] = 0.f;
      });
  if (it.is_seg) {
    constexpr int N = 4 / G > 0 ? 4 / G : 1;
    const int idx0 = group_reduce_scatter<LPG, 4>(acc, lane);
    if (group_owner<LPG, 4>(lane)) {
      float t[N];
#pragma unroll
      for (int c = 0; c < N; ++c) t[c] = acc[c];
      if (finish) hf_store<N>(At.partials + (int64_t)it.row * ISP_PARTIAL_TILE, (unsigned)(col - k_base + idx0) * 4u, t);
      else store_vec<N>(out + (int64_t)it.row * ldo + idx0, t);
    }
    if constexpr (FINISH) {
      if (hf_last(At, H, 0, lane)) {
        float t[4];
        hf_sum<LPG, 8>(At, H, (unsigned)(col - k_base) * 4u, lane, t);
        if (g == 0) store_vec<4>(dX + (int64_t)it.src_row * lddx + col, t);
      }
    }
    return;
  }
  if constexpr (G > 1) {
    const unsigned long long m_end = __ballot(ended), m_mid = __ballot(R.mid);
    const unsigned long long m_head = m_end & m_mid;
    if (m_head == 0) return;
    wave_lds_sync();
    float* __restrict__ tail = reinterpret_cast<float*>(L.ent);
#pragma unroll
    for (int v = 0; v < 4; ++v) tail[lane * 4 + v] = acc[v];
    wave_lds_sync();
    if ((m_head >> lane) & 1ull) {
      int j = lane - LPG;
      for (;;) {
#pragma unroll
        for (int v = 0; v < 4; ++v) head[v] += tail[j * 4 + v];
        if (((m_end >> j) & 1ull) || !((m_mid >> j) & 1ull)) break;
        j -= LPG;
      }
      store_vec<4>(out + (int64_t)L.dst[R.k] * ldo, head);
    }
  }
}

// live[q] = 1 for every entry q of the transpose whose source position p = perm[q] arg names (positions
// outside [0, nnz) - the -1 of empty rows, or anything a caller's array may hold - are ignored); live was
// zeroed before.  A row's columns name positions inside that row, so the lookups in inv_perm stay local.
__global__ void __launch_bounds__(256) k_mark_selected(const int32_t* __restrict__ arg, int64_t n, int64_t nnz,
                                                       const int32_t* __restrict__ inv_perm,
                                                       uint8_t* __restrict__ live) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const int32_t p = arg[t];
  if (p >= 0 && p < nnz) live[inv_perm[p]] = 1;
}

__global__ void __launch_bounds__(256) k_zero_u32(uint32_t* __restrict__ a, int64_t n) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) a[t] = 0u;
}

template <int VEC>
__global__ void __launch_bounds__(ISP_WG) k_sum_fixup(isp_view A, int d, int k0, float* __restrict__ Y, int64_t ldy) {
  hub_fixup<VEC, 1, false>(A, d, k0, Y, ldy);
}

__global__ void __launch_bounds__(ISP_WG) k_sum_fixup_wg(isp_view A, int d, int k0, float* __restrict__ Y, int64_t ldy) {
  hub_fixup_wg<4, 1, false>(A, d, k0, Y, ldy, 0);
}

bool aligned(const void* p, size_t a) { return ((uintptr_t)p & (a - 1)) == 0; }

unsigned item_grid(const isp_view& v) { return (unsigned)((v.n_blocks + v.n_seg + ISP_WAVES_PER_WG - 1) / ISP_WAVES_PER_WG); }
unsigned hub_grid(const isp_view& v) { return (unsigned)((v.n_hub + ISP_WAVES_PER_WG - 1) / ISP_WAVES_PER_WG); }

template <int VEC, int MODE>
isp_status fwd_tile(const isp_csr* A, const float* X, int64_t ldx, int d, int k0, float* Y, int64_t ldy, int32_t* arg,
                    hipStream_t s) {
  const isp_view& v = A->v;
  if (v.n_blocks + v.n_seg > 0) {
    if (v.values) k_reduce_fwd<VEC, MODE, true><<<item_grid(v), ISP_WG, 0, s>>>(v, v.indptr, v.indices, v.values, X, ldx, d, k0, Y, ldy, arg);
    else k_reduce_fwd<VEC, MODE, false><<<item_grid(v), ISP_WG, 0, s>>>(v, v.indptr, v.indices, v.values, X, ldx, d, k0, Y, ldy, arg);
    ISP_LAUNCH_CHECK();
  }
  if (v.n_hub > 0) {
    k_reduce_fixup<VEC, MODE><<<hub_grid(v), ISP_WG, 0, s>>>(v, d, k0, Y, ldy, arg);
    ISP_LAUNCH_CHECK();
  }
  return ISP_OK;
}

template <int LPG, int MODE>
isp_status minmax_grouped_tile(const isp_csr* A, const float* X, int64_t ldx, int d, int k_base, float* Y,
                               int64_t ldy, int32_t* arg, hipStream_t s) {
  const isp_view& v = A->v;
  const bool finish = hf_minmax_pays(A, v, LPG);
  const int n_items = v.n_blocks + v.n_seg;
  if (n_items > 0) {
    const unsigned grid = (unsigned)((n_items + ISP_WAVES_PER_WG - 1) / ISP_WAVES_PER_WG);
    if (finish) k_minmax_grouped<LPG, MODE, true><<<grid, ISP_WG, 0, s>>>(v, v.indptr, v.indices, v.values, X, ldx, d, k_base, Y, ldy, arg);
    else k_minmax_grouped<LPG, MODE, false><<<grid, ISP_WG, 0, s>>>(v, v.indptr, v.indices, v.values, X, ldx, d, k_base, Y, ldy, arg);
    ISP_LAUNCH_CHECK();
  }
  if (v.n_hub > 0 && !finish) {
    k_reduce_fixup<2, MODE><<<hub_grid(v), ISP_WG, 0, s>>>(v, d, k_base, Y, ldy, arg);
    ISP_LAUNCH_CHECK();
  }
  return ISP_OK;
}

template <int MODE>
isp_status fwd_all(const isp_csr* A, const float* X, int64_t ldx, int d, float* Y, int64_t ldy, int32_t* arg,
                   hipStream_t s) {
  const isp_view& av = A->v;
  if constexpr (MODE != R_MEAN) {
    // grouped kernel: 32-bit gather offsets, the partition within the LDS tables' limits
    const bool a32 = av.n_cols < (1 << 24) && ldx * 4 < (1 << 24) &&
                     ((uint64_t)av.n_cols * (uint64_t)ldx + (uint64_t)d) * 4u < ((uint64_t)1 << 32);
    const bool ok = av.nnz > 0 && a32 && d >= 4 && A->info.block_cost <= GS_MAX_ROWS &&
                    A->info.block_cost + av.hub_t <= GS_MAX_ENT && av.seg_len <= GS_MAX_ENT && !A->tune.no_grouped;
    if (ok) {
      // 128 columns per launch (a hub partial row holds 128 values and 128 positions), in one slice at every size.  Two
      // 64-column slices, measured with this kernel (us, one / two): 128 columns 2.4 M rows, 124 M entries 5715 / 5267, 800 k, 40 M
      // 1579 / 1579, 233 k, 115 M 2770 / 3105; 100 columns 5660 / 6700, 1546 / 1889, 2737 / 3417: they would pay for whole-line
      // rows of an operand far larger than the L2s alone, as for the sum.  Fewer workgroups per compute unit (15,000 bytes
      // more LDS each), which pay for the sum on its packed layout, lose in either form (one slice: 5923, 1837, 3944).
      isp_status st = ISP_OK;
      for (int k0 = 0; k0 < d && st == ISP_OK; k0 += 2 * ISP_WAVE) {
        const int k_base = d - k0 < 4 ? d - 4 : k0;  // (no launch narrower than a float4 lane)
        const int w = d - k_base < 2 * ISP_WAVE ? d - k_base : 2 * ISP_WAVE;
        // Four lanes to a row of up to 16 columns from 512 Ki entries (us with 8 / 4, max, 8 columns, R-MAT: 3 k rows, 30 k entries 10.1 / 10.5; 10 k, 100 k: 11.2 /
        // 11.7; 20 k, 300 k: 15.4 / 15.0; 60 k, 600 k: 18.7 / 17.6; 100 k, 1 M: 25.2 / 23.1; 60 k, 2.8 M: 41.9 / 38.3; 200 k, 8 M: 103 / 92; 230 k, 60 M: 623 / 545;
        // uniform, 100 k, 1 M 15.8 / 12.6, 500 k, 8 M: 117.7 / 114.2).
        if (w <= 16 && av.nnz >= (512 << 10)) st = minmax_grouped_tile<4, MODE>(A, X, ldx, d, k_base, Y, ldy, arg, s);
        else if (w <= 32) st = minmax_grouped_tile<8, MODE>(A, X, ldx, d, k_base, Y, ldy, arg, s);
        else if (w <= 64) st = minmax_grouped_tile<16, MODE>(A, X, ldx, d, k_base, Y, ldy, arg, s);
        else st = minmax_grouped_tile<32, MODE>(A, X, ldx, d, k_base, Y, ldy, arg, s);
      }
      return st;
    }
  }
  // min / max keep (value, position) pairs in the hub partial rows, so their column tiles stop at 128
  const bool v2 = d % 2 == 0 && ldx % 2 == 0 && ldy % 2 == 0 && aligned(X, 8) && aligned(Y, 8) && d > ISP_WAVE;
  isp_status st = ISP_OK;
  for (int k0 = 0; k0 < d && st == ISP_OK; k0 += (v2 ? 2 : 1) * ISP_WAVE)
    st = v2 ? fwd_tile<2, MODE>(A, X, ldx, d, k0, Y, ldy, arg, s) : fwd_tile<1, MODE>(A, X, ldx, d, k0, Y, ldy, arg, s);
  return st;
}

template <int LPG>
isp_status select_grouped_tile(const isp_csr* A, const int32_t* inv_perm, const float* dY, int64_t lddy, const int32_t* arg,
                               int d, int k_base, float* dX, int64_t lddx, hipStream_t s) {
  const isp_csr* At = A->At;
  const isp_view &v = At->v, &va = A->v;
  const bool finish = hf_pays(At, v, LPG);
  const int64_t words = (v.nnz + 3) / 4;
  k_zero_u32<<<(unsigned)((words + 255) / 256), 256, 0, s>>>(reinterpret_cast<uint32_t*>(At->sel_flags), words);
  ISP_LAUNCH_CHECK();
  if (va.n_blocks + va.n_hub > 0) {
    const unsigned grid = (unsigned)((va.n_blocks + va.n_hub + ISP_WAVES_PER_WG - 1) / ISP_WAVES_PER_WG);
    k_mark_lanes<LPG><<<grid, ISP_WG, 0, s>>>(va, va.indptr, arg, d, k_base, inv_perm, At->sel_flags);
    ISP_LAUNCH_CHECK();
  }
  if (v.n_blocks + v.n_seg > 0) {
    const unsigned grid = (unsigned)((v.n_blocks + v.n_seg + SELECT_WAVES - 1) / SELECT_WAVES);
    constexpr int WG = SELECT_WAVES * ISP_WAVE;
#define ISP_GO(HV, FN)                                                                                                       \
  k_select_grouped<LPG, HV, FN><<<grid, WG, 0, s>>>(v, v.indptr, v.indices, v.values, At->perm, At->sel_flags, dY, lddy, arg, d, \
                                                    k_base, dX, lddx)
    if (v.values) { if (finish) ISP_GO(true, true); else ISP_GO(true, false); }
    else { if (finish) ISP_GO(false, true); else ISP_GO(false, false); }
#undef ISP_GO
    ISP_LAUNCH_CHECK();
  }
  if (v.n_hub > 0 && !finish) {
    const int d_hi = d < k_base + 4 * LPG ? d : k_base + 4 * LPG;
    // (an alias of a handle whose launches finish their hub rows adds in their order)
    if (hf_few(At, v)) k_sum_fixup_wg<<<(unsigned)v.n_hub, ISP_WG, 0, s>>>(v, d_hi, k_base, dX, lddx);
    else k_sum_fixup<4><<<hub_grid(v), ISP_WG, 0, s>>>(v, d_hi, k_base, dX, lddx);
    ISP_LAUNCH_CHECK();
  }
  return ISP_OK;
}

template <class P, int VEC>
isp_status bwd_tile(const isp_csr* At, const typename P::args& pa, int d, int k0, float* dX, int64_t lddx,
                    hipStream_t s) {
  const isp_view& v = At->v;
  if (v.n_blocks + v.n_seg > 0) {
    k_reduce_bwd<P><<<item_grid(v), ISP_WG, 0, s>>>(v, v.indptr, v.indices, v.values, pa, d, k0, dX, lddx);
    ISP_LAUNCH_CHECK();
  }
  if (v.n_hub > 0) {
    k_sum_fixup<VEC><<<hub_grid(v), ISP_WG, 0, s>>>(v, d, k0, dX, lddx);
    ISP_LAUNCH_CHECK();
  }
  return ISP_OK;
}

template <int VEC, bool HV>
isp_status mean_bwd(const isp_csr* A, const float* dY, int64_t lddy, int d, int k0, float* dX, int64_t lddx,
                    hipStream_t s) {
  using P = mean_bwd_policy<VEC, HV>;
  typename P::args pa{{dY}, {lddy}, A->v.indptr, nullptr};
  return bwd_tile<P, VEC>(A->At, pa, d, k0, dX, lddx, s);
}

template <int VEC, bool HV>
isp_status select_bwd(const isp_csr* A, const float* dY, int64_t lddy, const int32_t* arg, int d, int k0, float* dX,
                      int64_t lddx, hipStream_t s) {
  using P = select_bwd_policy<VEC, HV>;
  typename P::args pa{{dY, reinterpret_cast<const float*>(arg)}, {lddy, (int64_t)d}, A->At->perm, A->At->sel_flags};
  return bwd_tile<P, VEC>(A->At, pa, d, k0, dX, lddx, s);
}

}  // namespace

isp_status isp_spmm_reduce_launch(const isp_csr* A, const float* X, int64_t ldx, int32_t d, int reduce, float* Y,
                                  int64_t ldy, int32_t* arg, hipStream_t s) {
  if (reduce == R_MEAN) {  // the tuned kernel divides each finished row by its length
    bool done = false;
    const isp_status st = isp_spmm_grouped_launch(A, X, ldx, d, Y, ldy, 1, nullptr, s, &done);
    if (done || st != ISP_OK) return st;
    return fwd_all<R_MEAN>(A, X, ldx, d, Y, ldy, arg, s);
  }
  if (reduce == R_MIN) return fwd_all<R_MIN>(A, X, ldx, d, Y, ldy, arg, s);
  return fwd_all<R_MAX>(A, X, ldx, d, Y, ldy, arg, s);
}

isp_status isp_spmm_reduce_bwd_launch(isp_csr* A, const float* dY, int64_t lddy, int32_t d, int reduce,
                                      const int32_t* arg, float* dX, int64_t lddx, hipStream_t s) {
  const isp_csr* At = A->At;
  if (reduce == R_MEAN && At->v.nnz > 0) {
    // the tuned kernels on A^T with every value divided by its source row's length (computed once per handle)
    const float *mv = nullptr, *mv_packed = nullptr;
    isp_status st = isp_transpose_mean_values(A, s, &mv, &mv_packed);
    if (st != ISP_OK) return st;
    bool done = false;
    st = isp_spmm_grouped_launch(At, dY, lddy, d, dX, lddx, 0, mv, s, &done, mv_packed);
    if (done || st != ISP_OK) return st;
  }
  const bool hv = At->v.values != nullptr;
  const bool v2 = d % 2 == 0 && lddy % 2 == 0 && lddx % 2 == 0 && aligned(dY, 8) && aligned(dX, 8) &&
                  aligned(arg, 8) && d > ISP_WAVE;
  isp_status st = ISP_OK;
  const isp_view& tv = At->v;
  const int32_t* inv_perm = nullptr;
  if (reduce != R_MEAN && tv.nnz > 0 && (st = isp_transpose_inverse_perm(A, s, &inv_perm)) != ISP_OK) return st;
  auto fits = [&](int64_t ld) {  // 32-bit gather offsets into a matrix of A's rows
    return tv.n_cols < (1 << 24) && ld * 4 < (1 << 24) && ((uint64_t)tv.n_cols * (uint64_t)ld + (uint64_t)d) * 4u < ((uint64_t)1 << 32);
  };
  auto items_fit = [](const isp_csr* M) {
    return M->info.block_cost <= GS_MAX_ROWS && M->info.block_cost + M->v.hub_t <= GS_MAX_ENT && M->v.seg_len <= GS_MAX_ENT;
  };
  if (reduce != R_MEAN && tv.nnz > 0 && d >= 4 && fits(lddy) && fits(d) && items_fit(A) && items_fit(At) && !At->tune.no_grouped) {
    for (int k0 = 0; k0 < d && st == ISP_OK; k0 += ISP_PARTIAL_TILE) {
      const int k_base = d - k0 < 4 ? d - 4 : k0;  // (no launch narrower than a float4 lane)
      const int w = d - k_base < ISP_PARTIAL_TILE ? d - k_base : ISP_PARTIAL_TILE;
      if (select_four_lanes(w, A->v.nnz, A->At->v.n_hub)) st = select_grouped_tile<4>(A, inv_perm, dY, lddy, arg, d, k_base, dX, lddx, s);
      else if (w <= 32) st = select_grouped_tile<8>(A, inv_perm, dY, lddy, arg, d, k_base, dX, lddx, s);
      else if (w <= 64) st = select_grouped_tile<16>(A, inv_perm, dY, lddy, arg, d, k_base, dX, lddx, s);
      else if (w <= 128) st = select_grouped_tile<32>(A, inv_perm, dY, lddy, arg, d, k_base, dX, lddx, s);
      else st = select_grouped_tile<64>(A, inv_perm, dY, lddy, arg, d, k_base, dX, lddx, s);
    }
    return st;
  }
  if (reduce != R_MEAN && tv.nnz > 0) {  // which entries of A does arg name at all (any column)?
    const int64_t words = (tv.nnz + 3) / 4, n_arg = A->v.n_rows * (int64_t)d;
    k_zero_u32<<<(unsigned)((words + 255) / 256), 256, 0, s>>>(reinterpret_cast<uint32_t*>(At->sel_flags), words);
    ISP_LAUNCH_CHECK();
    if (n_arg > 0) {
      k_mark_selected<<<(unsigned)((n_arg + 255) / 256), 256, 0, s>>>(arg, n_arg, tv.nnz, inv_perm, At->sel_flags);
      ISP_LAUNCH_CHECK();
    }
  }
  for (int k0 = 0; k0 < d && st == ISP_OK; k0 += (v2 ? 2 : 1) * ISP_WAVE) {
    if (reduce == R_MEAN) {
      if (v2 && hv) st = mean_bwd<2, true>(A, dY, lddy, d, k0, dX, lddx, s);
      else if (v2) st = mean_bwd<2, false>(A, dY, lddy, d, k0, dX, lddx, s);
      else if (hv) st = mean_bwd<1, true>(A, dY, lddy, d, k0, dX, lddx, s);
      else st = mean_bwd<1, false>(A, dY, lddy, d, k0, dX, lddx, s);
    } else {
      if (v2 && hv) st = select_bwd<2, true>(A, dY, lddy, arg, d, k0, dX, lddx, s);
      else if (v2) st = select_bwd<2, false>(A, dY, lddy, arg, d, k0, dX, lddx, s);
      else if (hv) st = select_bwd<1, true>(A, dY, lddy, arg, d, k0, dX, lddx, s);
      else st = select_bwd<1, false>(A, dY, lddy, arg, d, k0, dX, lddx, s);
    }
  }
  return st;
}
