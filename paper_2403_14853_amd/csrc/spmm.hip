// SpMM, sum reduction: Y = A X with A in CSR and X dense row-major (paper: abstract, Sections 1,
// 3.4, 3.5).  The backward dX = A^T dY is this same code run on the cached transpose's handle
// (Section 3.3).  Gather-bound: per nonzero one 4*d-byte row of X is fetched and d FMAs are done,
// so the kernels are built around coalesced row gathers, not around matrix cores.
#include "hub_finish.h"
#include "output_rule.h"
#include "run_stream.h"
#include "stage_rule.h"

namespace {
using namespace isp_dev;

template <int VEC_, int T_, bool HAS_VAL_>
struct spmm_policy {
  static constexpr int VEC = VEC_, T = T_, NG = 1;
  static constexpr int U = (VEC * T >= 4) ? 4 : 8;
  static constexpr bool HAS_VAL = HAS_VAL_, ACCUMULATE = false, NEEDS_PERM = false, HAS_FINISH = false;
  struct args { const float* src[1]; int64_t ld[1]; };
  struct row_state {};
  __device__ static inline void row_begin(const args&, row_state&, int, const int (&)[T], const bool (&)[T]) {}
  __device__ static inline void edge(const args&, row_state&, float a, const float (&x)[1][T][VEC],
                                     float (&acc)[T][VEC], const bool (&)[T], const edge_info&) {
#pragma unroll
    for (int tt = 0; tt < T; ++tt)
#pragma unroll
      for (int v = 0; v < VEC; ++v) acc[tt][v] = fmaf(a, x[0][tt][v], acc[tt][v]);
  }
};

template <int VEC, int T, bool HAS_VAL>
__global__ void __launch_bounds__(ISP_WG) k_spmm(isp_view A, const int64_t* __restrict__ indptr,
                                                 const int32_t* __restrict__ indices,
                                                 const float* __restrict__ values, const float* __restrict__ X,
                                                 int64_t ldx, int d, int k0, float* __restrict__ Y, int64_t ldy) {
  using P = spmm_policy<VEC, T, HAS_VAL>;
  typename P::args pa;
  pa.src[0] = X;
  pa.ld[0] = ldx;
  stream_item<P>(A, indptr, indices, values, pa, d, k0, Y, ldy);
}

// One workgroup per hub row.
template <int VEC, int T>
__global__ void __launch_bounds__(ISP_WG) k_spmm_fixup(isp_view A, int d, int k0, float* __restrict__ Y, int64_t ldy,
                                                       int split_above) {
  hub_fixup_wg<VEC, T, false>(A, d, k0, Y, ldy, split_above);
}
// Pieces of the packed layout: rows of up to this many are added by one wavefront.
constexpr int PACKED_SPLIT = 32;

// Mean reduction: the fixed-order sum of a hub row's segments, divided by the row's length.
__global__ void __launch_bounds__(ISP_WG) k_spmm_fixup_mean(isp_view A, int d, int k0, float* __restrict__ Y,
                                                            int64_t ldy, int split_above) {
  hub_fixup_wg<4, 1, true>(A, d, k0, Y, ldy, split_above);
}

template <int VEC, int T>
isp_status launch_tile(const isp_csr* A, const float* X, int64_t ldx, int d, int k0, float* Y, int64_t ldy,
                       hipStream_t s) {
  const isp_view& v = A->v;
  const int n_items = v.n_blocks + v.n_seg;
  if (n_items > 0) {
    const unsigned grid = (unsigned)((n_items + ISP_WAVES_PER_WG - 1) / ISP_WAVES_PER_WG);
    if (v.values)
      k_spmm<VEC, T, true><<<grid, ISP_WG, 0, s>>>(v, v.indptr, v.indices, v.values, X, ldx, d, k0, Y, ldy);
    else
      k_spmm<VEC, T, false><<<grid, ISP_WG, 0, s>>>(v, v.indptr, v.indices, v.values, X, ldx, d, k0, Y, ldy);
    ISP_LAUNCH_CHECK();
  }
  if (v.n_hub > 0) {
    k_spmm_fixup<VEC, T><<<(unsigned)v.n_hub, ISP_WG, 0, s>>>(v, d, k0, Y, ldy, 0);
    ISP_LAUNCH_CHECK();
  }
  return ISP_OK;
}


// ---- run-streaming fast path (run_stream.h) --------------------------------------------------------
// LPG lanes x float4 cover one slice of 4 * LPG feature columns; G = 64 / LPG nonzeros per gather
// instruction.  Slice s of tile k_base covers columns [k_base + s * 4 * LPG, +4 * LPG).
// ADDR32: every byte offset into X fits 32 bits and both factors of column * row-pitch fit 24 bits, so
// the gather address is one full-rate 24-bit multiply-add on top of a scalar base pointer.
// MEAN: finished rows are divided by their length (partial rows are not: their fix-up divides).
// FINISH: hub rows are put together here (hub_finish.h).  A kernel of its own: launches that have none to finish ran 2 % longer
// with that code in them (4 k rows, 37 k entries 4.41 -> 4.53 us).
// STREAM: what is written past the caches: STREAM_ROWS: rows of Y that an item finishes (output_rule.h; never with the small LDS tables, whose operand the L2s
// hold), STREAM_PIECES: the packed layout's partial rows.  Kernels of their own as well: with the choice at run time the small launch took 4.47 us.
constexpr int SPMM_RING = 4;
constexpr int STREAM_ROWS = 1, STREAM_PIECES = 2;

// On the packed layout, launches that gather more than three and a half lines of a row ask for LDS they do not use, so that a
// compute unit holds four workgroups instead of five: the rows of X that the whole chip has in flight and in use at a time then
// fit the L2s better.  With fewer lines the latency counts.  us per SpMM with five / four (/ three):
//   4 lines and more: 233 k columns, 115 M entries: 128 columns 2518 / 2440 / 2599, 256 5069 / 4905 / 5219, 97 2347 / 2335; 2.4 M, 124 M: 128 4755 /
//   4672 / 4804, 100 4832 / 4774; 200 k, 20 M: 128 565 / 549 / 566; 800 k, 40 M: 100 1437 / 1418; 400 k, 12 M: 200 1019 / 985;
//   3.75 and 3.9 (92 and 94 columns, ragged): 400 k, 12 M: 442 / 431, 463 / 449; 1 M, 20 M: 847 / 829, 875 / 861;
//   3.5 (84, 88 columns, ragged): 233 k, 115 M: 2105 / 2145, 2110 / 2149; 2.4 M, 124 M: 88 4117 / 4109; 500 k, 10 M: 88 384 / 376;
//   3 to 3.1 (65 to 96): 233 k, 115 M: 69 1956 / 2035, 96 1949 / 2043; 139 k, 43 M: 69 734 / 771; 800 k, 40 M: 72 1028 / 1049, 96 1058 / 1078; 2.4 M,
//   124 M: 96 3514 / 3572; 80 k, 12 M: 96 222 / 232; copies of 90 columns (96 floats): 233 k 1984 / 2075;
//   2 (64 columns): 2326 / 2325;  1 (32): 1213 / 1248.
constexpr unsigned SPMM_FOUR_PER_CU = 160 * 1024 / 4 - sizeof(rn_lds);

template <int LPG, bool ADDR32, int VEC, bool MEAN, bool FINISH, int CAP = GS_MAX_ENT, int STREAM = 0>
__global__ void __launch_bounds__(ISP_WG) k_spmm_grouped(
    isp_view A, const int64_t* __restrict__ indptr, const int32_t* __restrict__ indices,
    const float* __restrict__ values, const float* __restrict__ X, int64_t ldx, int d, int k_base, int n_slices,
    float* __restrict__ Y, int64_t ldy) {
  constexpr int G = ISP_WAVE / LPG;
  __shared__ rn_lds_of<CAP> lds;
  const int lane = threadIdx.x & (ISP_WAVE - 1);
  const int w = threadIdx.x >> 6;
  const int slice = __builtin_amdgcn_readfirstlane((int)(blockIdx.x % n_slices));
  const int item = __builtin_amdgcn_readfirstlane((int)(blockIdx.x / n_slices) * ISP_WAVES_PER_WG + w);
  if (item >= A.n_blocks + A.n_seg) return;
  const item_range it = locate_item(A, indptr, item);
  if (it.skip) return;
  auto& L = lds.w[w];
  // Rows of a derived matrix (packed layout) beyond the real ones are pieces of long rows: like a hub segment
  // each adds into a partial row, named by piece_slot.  A block never mixes real rows and pieces.
  const bool pieces = !it.is_seg && (int64_t)it.row >= A.n_real_rows;
  const bool to_partial = it.is_seg || pieces;
  const bool finish = FINISH && it.is_seg;
  hub_ref H{0, 0, 0};
  if (finish) H.h = A.seg_hub[it.row];
  const rn_run R = rn_prepare<G>(it, indptr, indices, values,
                                 pieces ? A.piece_slot - A.n_real_rows : nullptr, L, lane);

  if (finish) {
    H.s0 = A.hub_seg_ptr[H.h];
    H.s1 = A.hub_seg_ptr[H.h + 1];
  }
  const int g = lane / LPG, q = lane % LPG;
  int col = k_base + (slice * LPG + q) * VEC;
  const bool lane_on = col < d;
  // (lanes past d work on the last columns again: every step is one load per lane without a branch, from a line
  // that the row's gather touches anyway, and they store what the columns' own lane stores)
  col = k_base + tail_col<VEC>(col - k_base, d - k_base);
  const float* __restrict__ xcol = X + col;
  const unsigned lane_byte = (unsigned)col * 4u;
  const unsigned pitch_byte = (unsigned)ldx * 4u;
  float* __restrict__ out = to_partial ? A.partials + (col - k_base) : Y + col;
  const unsigned ldo = to_partial ? (unsigned)ISP_PARTIAL_TILE : (unsigned)ldy;  // (the launcher checks that it fits)
  auto row_of = [&](int dst) { return out + (uint64_t)(unsigned)dst * ldo; };
  auto put = [&](int dst, const float (&o)[VEC]) {
    if constexpr (VEC == 4 && STREAM != 0) {
      if (STREAM == (STREAM_ROWS | STREAM_PIECES) || to_partial == (STREAM == STREAM_PIECES)) {
        store_vec4_nt(row_of(dst), o);
        return;
      }
    }
    store_vec<VEC>(row_of(dst), o);
  };

  float acc[VEC], head[VEC], x[SPMM_RING][VEC];
#pragma unroll
  for (int v = 0; v < VEC; ++v) acc[v] = head[v] = 0.f;
  if (!to_partial)  // the empty rows' outputs (also their mean); a piece is never empty
    for (int i = g; i < R.n_empty; i += G) put(L.dst[RN_EMPTY0 - i], acc);

  bool carried = R.mid;  // the next row to end began in an earlier run
  bool ended = false;    // a row has ended in this run
  auto inv_len = [&](int k) { return 1.f / (float)((int)L.end[k] - (k > 0 ? (int)L.end[k - 1] : 0)); };
  rn_stream<SPMM_RING, true, false>(
      L, R,
      [&](int u, int c, int, int, bool) {
        if constexpr (ADDR32) {
          const unsigned off = __umul24((unsigned)c, pitch_byte) + lane_byte;
          load_vec<VEC>(reinterpret_cast<const float*>(reinterpret_cast<const char*>(X) + off), x[u]);
        } else {
          load_vec<VEC>(xcol + (int64_t)c * ldx, x[u]);
        }
      },
      [&](int u, float a, int) {
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] = fmaf(a, x[u][v], acc[v]);
      },
      [&](int k, int row) {
#pragma unroll
        for (int v = 0; v < VEC; ++v)
          if (carried) head[v] = acc[v];  // (as a choice between the two the scalar-lane kernel kept them in memory)
        if (!carried) {
          if (MEAN && !to_partial) {
            const float inv = inv_len(k);
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[v] *= inv;
          }
          put(row, acc);
        }
        carried = false;
        ended = true;
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] = 0.f;
      });

  if (it.is_seg) {  // one row: the groups' sums, spread over the groups (this lane stores R columns from idx0 on)
    constexpr int N = VEC / G > 0 ? VEC / G : 1;
    const int idx0 = group_reduce_scatter<LPG, VEC>(acc, lane);
    if (group_owner<LPG, VEC>(lane) && lane_on) {
      float t[N];
#pragma unroll
      for (int c = 0; c < N; ++c) t[c] = acc[c];
      if (finish) hf_store<N>(A.partials + (int64_t)it.row * ISP_PARTIAL_TILE, (unsigned)(col - k_base + idx0) * 4u, t);
      else store_vec<N>(row_of(it.row) + idx0, t);
    }
    if constexpr (FINISH) {
      if (hf_last(A, H, slice, lane)) {
        float t[4];
        hf_sum<LPG, CAP == GS_MAX_ENT ? 16 : 8>(A, H, (unsigned)(col - k_base) * 4u, lane, t);
        if (MEAN) {
          const float inv = A.inv_len[it.src_row];
#pragma unroll
          for (int v = 0; v < 4; ++v) t[v] *= inv;
        }
        if (g == 0 && lane_on) store_vec<4>(Y + (int64_t)it.src_row * ldy + col, t);
      }
    }
    return;
  }
  if constexpr (G > 1) {
    // rows cut by a run boundary: the run in which such a row ends adds the earlier runs' last, unfinished sums
    const unsigned long long m_end = __ballot(ended), m_mid = __ballot(R.mid);
    const unsigned long long m_head = m_end & m_mid;
    if (m_head == 0) return;
    wave_lds_sync();  // (every entry has been read)
    float* __restrict__ tail = reinterpret_cast<float*>(L.ent);
#pragma unroll
    for (int v = 0; v < VEC; ++v) tail[lane * VEC + v] = acc[v];
    wave_lds_sync();
    if ((m_head >> lane) & 1ull) {
      int j = lane - LPG;
      for (;;) {
#pragma unroll
        for (int v = 0; v < VEC; ++v) head[v] += tail[j * VEC + v];
        if (((m_end >> j) & 1ull) || !((m_mid >> j) & 1ull)) break;  // the row began in that run
        j -= LPG;
      }
      if (MEAN && !to_partial) {
        const float inv = inv_len(R.k);
#pragma unroll
        for (int v = 0; v < VEC; ++v) head[v] *= inv;
      }
      put(L.dst[R.k], head);
    }
  }
}

template <int LPG, int VEC = 4>
isp_status launch_grouped(const isp_csr* A, const float* X, int64_t ldx, int d, int k_base, int n_slices, float* Y,
                          int64_t ldy, int mean_mode, const float* values_override, hipStream_t s,
                          const float* values_override_packed = nullptr) {
  // The packed layout (a derived matrix in which the pieces of long rows share work items) when the handle has
  // one; an override of the values is in the order of A's own entries and therefore runs on A's own partition.
  const bool packed = A->has_packed && (!values_override || values_override_packed) &&
                      A->packed_block_cost + A->vp.hub_t <= GS_MAX_ENT &&
                      A->packed_block_cost / A->packed_row_cost <= GS_MAX_ROWS;
  const isp_view& v = packed ? A->vp : A->v;
  const int width = n_slices * LPG * VEC < d - k_base ? n_slices * LPG * VEC : d - k_base;
  const bool a32 = v.n_cols < (1 << 24) && ldx * 4 < (1 << 24) &&
                   ((uint64_t)v.n_cols * (uint64_t)ldx + (uint64_t)d) * 4u < ((uint64_t)1 << 32);
  const bool finish = VEC == 4 && a32 && n_slices <= HF_SLICES && hf_pays(A, v, LPG);  // (else a fix-up launch adds the hub rows)
  const bool stream = streams_output(v.n_real_rows, d), stream_pieces = packed && streams_pieces(A->info.spmm_pieces, width);
  // (one value per stored entry, in the order of the view's entries)
  const float* vals = values_override ? (packed ? values_override_packed : values_override) : v.values;
  const int n_items = v.n_blocks + v.n_seg;
  if (n_items > 0) {
    const unsigned grid = (unsigned)((n_items + ISP_WAVES_PER_WG - 1) / ISP_WAVES_PER_WG) * (unsigned)n_slices;
    const unsigned spare = packed && 2 * isp_stage::line_sum((uintptr_t)(X + k_base), ldx, width) > 7 * isp_stage::ALIGN
                               ? SPMM_FOUR_PER_CU : 0u;
#define ISP_GO2(A32, MN, FN, ST)                                                                                    \
  k_spmm_grouped<LPG, A32, VEC, MN, FN, GS_MAX_ENT, ST><<<grid, ISP_WG, spare, s>>>(v, v.indptr, v.indices, vals, X, ldx, d, \
                                                                                    k_base, n_slices, Y, ldy)
#define ISP_GO1(A32, MN, FN) do { if (stream) ISP_GO2(A32, MN, FN, A32 && VEC == 4 ? STREAM_ROWS : 0); else ISP_GO2(A32, MN, FN, 0); } while (0)
#define ISP_GO_PACKED(A32, MN)                                                                                         \
  do {                                                                                                              \
    if (stream) ISP_GO2(A32, MN, false, A32 && VEC == 4 ? STREAM_ROWS | STREAM_PIECES : 0);                            \
    else ISP_GO2(A32, MN, false, A32 && VEC == 4 ? STREAM_PIECES : 0);                                                 \
  } while (0)
#define ISP_GO(A32, MN) do { if (stream_pieces) ISP_GO_PACKED(A32, MN); else if (finish) ISP_GO1(A32, MN, A32 && VEC == 4); else ISP_GO1(A32, MN, false); } while (0)
    // (one group to a wavefront, 129 to 224 columns, has work for 14 per compute unit before seven at a time pay: 25 k columns,
    // 408 k entries, 208 columns (6.6 per unit) 31.4 us with five, 33.8 with seven; 17 k, 601 k: 176 (8.5) 34.7 / 36.7; 23 k, 1 M: 135 (17.2)
    // 51.2 / 46.8; 22 k, 862 k: 207 (14.8) 51.0 / 49.8)
    if (VEC == 4 && a32 && !packed && rn_small_tables(A, v, width, grid, LPG == ISP_WAVE ? 14 : 5)) {
#define ISP_SMALL1(MN, FN)                                                                                              \
  k_spmm_grouped<LPG, true, 4, MN, FN, RN_SMALL><<<grid, ISP_WG, 0, s>>>(v, v.indptr, v.indices, vals, X, ldx, d, k_base, \
                                                                     n_slices, Y, ldy)
#define ISP_SMALL(MN) do { if (finish) ISP_SMALL1(MN, true); else ISP_SMALL1(MN, false); } while (0)
      if (mean_mode == 1) ISP_SMALL(true); else ISP_SMALL(false);
#undef ISP_SMALL
#undef ISP_SMALL1
    } else if constexpr (VEC < 4) {  // scalar lanes are only dispatched with 32-bit addressing and for the plain sum
      ISP_GO(true, false);
    } else if (mean_mode == 1) {
      if (a32) ISP_GO(true, true); else ISP_GO(false, true);
    } else {
      if (a32) ISP_GO(true, false); else ISP_GO(false, false);
    }
#undef ISP_GO
#undef ISP_GO1
#undef ISP_GO2
#undef ISP_GO_PACKED
    ISP_LAUNCH_CHECK();
  }
  if (v.n_hub > 0 && !finish) {
    // the columns this launch covered: [k_base, min(d, k_base + n_slices * LPG * VEC))
    const int d_hi = (k_base + n_slices * LPG * VEC < d) ? k_base + n_slices * LPG * VEC : d;
    const int split = packed ? PACKED_SPLIT : 0;
    if (mean_mode == 1) k_spmm_fixup_mean<<<(unsigned)v.n_hub, ISP_WG, 0, s>>>(v, d_hi, k_base, Y, ldy, split);  // VEC = 4 only
    else k_spmm_fixup<VEC, 4 / VEC><<<(unsigned)v.n_hub, ISP_WG, 0, s>>>(v, d_hi, k_base, Y, ldy, split);
    ISP_LAUNCH_CHECK();
  }
  return ISP_OK;
}

bool aligned(const void* p, size_t a) { return ((uintptr_t)p & (a - 1)) == 0; }

// Copy of columns [k0, k0 + w) of X, row by row, to rows of `pitch` floats (what lies behind column w is never
// read).  32 lanes per row, of which the first ceil(w / 4) have work; the last one of a row that is no multiple of 4 moves back.
__global__ void __launch_bounds__(256) k_stage_cols(const float* __restrict__ X, int64_t ldx, int64_t n, int k0, int w,
                                                    int pitch, float* __restrict__ out) {
  const int q = threadIdx.x & 31;
  if (q * 4 >= w) return;
  const int c = tail_col<4>(q * 4, w);
  constexpr int R = 4;  // rows in flight per lane
  const int64_t r0 = (int64_t)blockIdx.x * (8 * R) + (threadIdx.x >> 5);
  float t[R][4];
#pragma unroll
  for (int u = 0; u < R; ++u)
    if (r0 + 8 * u < n) load_vec<4>(X + (r0 + 8 * u) * ldx + k0 + c, t[u]);
#pragma unroll
  for (int u = 0; u < R; ++u)
    if (r0 + 8 * u < n) store_vec<4>(out + (r0 + 8 * u) * pitch + c, t[u]);
}

}  // namespace

// The grouped fast path; *done = false (and nothing launched) when the operands do not qualify.
// mean_mode: see k_spmm_grouped.  values_override (optional): nnz values, in A's entry order, used in place of
// A's own (the backward of the mean reduction passes the transpose's values divided by the source rows' lengths).
isp_status isp_spmm_grouped_launch(const isp_csr* A, const float* X, int64_t ldx, int32_t d, float* Y, int64_t ldy,
                                   int mean_mode, const float* values_override, hipStream_t s, bool* done,
                                   const float* values_override_packed) {
  const isp_view& av = A->v;
  // float4 lanes at every width from 4 columns up and any alignment (the last lane of a row moves back where the
  // width is no multiple of 4); below, scalar lanes, only with 32-bit addressing and for the plain sum.
  const int vec = d >= 4 ? 4 : 1;
  const bool a32 = av.n_cols < (1 << 24) && ldx * 4 < (1 << 24) &&
                   ((uint64_t)av.n_cols * (uint64_t)ldx + (uint64_t)d) * 4u < ((uint64_t)1 << 32);
  // (a matrix without entries never reads X, which may then be absent: the generic path handles it)
  const bool grouped_ok = av.nnz > 0 && (vec == 4 || (a32 && mean_mode == 0)) && A->info.block_cost <= GS_MAX_ROWS &&
                          A->info.block_cost + av.hub_t <= GS_MAX_ENT && av.seg_len <= GS_MAX_ENT &&
                          ldy < ((int64_t)1 << 32) && !A->tune.no_grouped;
  *done = grouped_ok;
  if (!grouped_ok) return ISP_OK;
  if (vec < 4) return launch_grouped<4, 1>(A, X, ldx, d, 0, 1, Y, ldy, 0, values_override, s, values_override_packed);
  // float4 lanes: 4 / 8 / 16 / 32 / 64 lanes per group <-> column slices of 16 / 32 / 64 / 128 / 256 floats.  What
  // follows was measured on graphs of 37 k ... 124 M entries at widths 16 ... 301 (us, best of the shapes tried):
  //  - wide rows of whole lines are covered 128 columns at a time, each launch with the group that fits it, from 2 M
  //    entries up (2.4 M entries, 256 columns: 2 x 95 against 210 in one launch; 115 M entries, 160 columns:
  //    2509 + 771 against 4310), 256 at a time below (1.2 M entries, 192 columns: 72 against 77) and where rows
  //    start anywhere and are not copied (below): there every launch pays for the lines that its edges cut (602 columns:
  //    667 -> 620 on 2.4 M entries, 4931 -> 4584 on 16.9 M);
  //  - in a launch of up to 128 columns the smallest group that covers them wins (groups of 4 lanes, which share an
  //    instruction between 16 entries, only from 768 Ki entries up: they take longer to set an item up; us with 8 / 4 lanes, 8 and 16 columns,
  //    R-MAT: 10 k rows, 100 k entries 6.2 / 6.2, 6.1 / 6.1; 60 k, 600 k: 10.4 / 10.5, 10.3 / 10.7; 200 k, 800 k: 13.9 / 11.8, 14.6 / 13.1; 5 k, 800 k:
  //    12.5 / 10.8, 12.0 / 10.7; 100 k, 990 k: 14.5 / 13.0, 15.2 / 14.7; uniform, 30 k, 120 k 4.9 / 5.2, 5.1 / 5.2, 50 k, 900 k 8.8 / 8.2, 9.5 / 8.8);
  //  - 128 whole-line columns run as two 64-column slices, dealt to alternating XCDs, where the dense operand is far
  //    larger than an L2 (each L2 then keeps half-rows of twice as many hot columns): from 80 k columns up (60 k: 47 ->
  //    50), but with the packed layout, whose bands already fit, only from 512 k (233 k columns: 2509 -> 2665; 2.4 M:
  //    5144 -> 4731).  What it gives in between depends on where X is: 169 k columns (X and Y 87 MB each), one X and Y
  //    again and again, which the Infinity Cache holds, 108 -> 95; two pairs in turn 109 -> 108; four or more pairs in
  //    turn, X from HBM every time, 112 -> 113: the misses' rate decides there, whatever the L2s keep.  A layer's X
  //    has usually just been written;
  //  - between 129 and 256 columns in one launch, one 64-lane group up to 224 columns (but 128 columns and the rest
  //    from 512 k columns up: 200 columns, 4586 against 5021 on 233 k, 1608 against 1531 on 1 M), else two
  //    128-column slices.
  // ISP_SPMM_LPG / ISP_SPMM_TILE (read when the handle was built) override the choices for tuning.
  const bool packed = A->has_packed && (!values_override || values_override_packed);
  int tile = av.nnz >= 2000000 && ldx % 32 == 0 ? 128 : ISP_PARTIAL_TILE;
  const int64_t slice_cols = packed ? 512 << 10 : 80 << 10;
  // Are the columns of each launch copied to whole lines first?  (Rule and figures: stage_rule.h.)
  const bool stage = A->stages && d >= 4 &&
                     (A->tune.stage_min > 0 ? ldx % 32 != 0 || !aligned(X, 128)
                                           : isp_stage::call_pays({av.nnz, av.n_cols, ldx, d,
                                                                   isp_stage::operand_lines((uintptr_t)X, ldx, d, tile, av.n_cols),
                                                                   isp_stage::copied_lines(d), packed,
                                                                   av.n_cols >= slice_cols,
                                                                   packed ? 2 * (int64_t)A->info.spmm_cut_rows > av.n_rows : av.n_hub == 0}));
  if (stage || (A->stages && A->tune.stage_min > 0)) tile = isp_stage::COLS;  // (the latter for aligned X too: same launches)
  if (A->tune.spmm_tile) tile = A->tune.spmm_tile;
  // (a handle with the packed layout may keep its copies among the rows that launches on the other partition write)
  const bool place_free = packed || !A->has_packed;
  const bool slices = (ldx % 32 == 0 || stage) && av.n_cols >= slice_cols;
  isp_status st = ISP_OK;
  for (int k0 = 0, w; k0 < d && st == ISP_OK; k0 += w) {
    const int k_base = isp_stage::tile_start(k0, d);
    w = isp_stage::tile_width(k_base, d, tile, av.n_cols);
    int lpg = 32;
    if (w <= 16 && av.nnz >= (768 << 10)) lpg = 4;
    else if (w <= 32) lpg = 8;
    else if (w <= 64 || (w == 128 && slices)) lpg = 16;
    else if (w > 128 && w <= 224) lpg = 64;
    if (A->tune.spmm_lpg) lpg = A->tune.spmm_lpg;
    const int ns = (w + 4 * lpg - 1) / (4 * lpg);
    const float* Xt = X;  // what this launch gathers from
    int64_t ldt = ldx;
    // (a launch whose groups reach beyond w, which only the overrides make, gathers from X)
    if (stage && A->stage && place_free && isp_stage::pitch(w) <= A->stage_cols && (k_base + w == d || ns * 4 * lpg == w)) {
      ldt = isp_stage::pitch(w);
      k_stage_cols<<<(unsigned)((av.n_cols + 31) / 32), 256, 0, s>>>(X, ldx, av.n_cols, k_base, w, (int)ldt, A->stage);
      ISP_LAUNCH_CHECK();
      Xt = A->stage - k_base;
    }
    switch (lpg) {
      case 4: st = launch_grouped<4>(A, Xt, ldt, d, k_base, ns, Y, ldy, mean_mode, values_override, s, values_override_packed); break;
      case 8: st = launch_grouped<8>(A, Xt, ldt, d, k_base, ns, Y, ldy, mean_mode, values_override, s, values_override_packed); break;
      case 16: st = launch_grouped<16>(A, Xt, ldt, d, k_base, ns, Y, ldy, mean_mode, values_override, s, values_override_packed); break;
      case 32: st = launch_grouped<32>(A, Xt, ldt, d, k_base, ns, Y, ldy, mean_mode, values_override, s, values_override_packed); break;
      default: st = launch_grouped<64>(A, Xt, ldt, d, k_base, ns, Y, ldy, mean_mode, values_override, s, values_override_packed); break;
    }
  }
  return st;
}

isp_status isp_spmm_launch(const isp_csr* A, const float* X, int64_t ldx, int32_t d, float* Y, int64_t ldy,
                           hipStream_t s) {
  bool done = false;
  isp_status st0 = isp_spmm_grouped_launch(A, X, ldx, d, Y, ldy, 0, nullptr, s, &done);
  if (done || st0 != ISP_OK) return st0;
  // lanes-over-features layout: the widest vector the width and alignment allow
  int vec = 1;
  if (d > 2 * ISP_WAVE && d % 4 == 0 && ldx % 4 == 0 && ldy % 4 == 0 && aligned(X, 16) && aligned(Y, 16)) vec = 4;
  else if (d > ISP_WAVE && d % 2 == 0 && ldx % 2 == 0 && ldy % 2 == 0 && aligned(X, 8) && aligned(Y, 8)) vec = 2;
  isp_status st = ISP_OK;
  int k0 = 0;
  while (k0 < d && st == ISP_OK) {  // column tiles of at most ISP_PARTIAL_TILE floats
    const int w = d - k0;
    int step;
    if (vec == 4) { st = launch_tile<4, 1>(A, X, ldx, d, k0, Y, ldy, s); step = 4 * ISP_WAVE; }
    else if (vec == 2 && w <= 2 * ISP_WAVE) { st = launch_tile<2, 1>(A, X, ldx, d, k0, Y, ldy, s); step = 2 * ISP_WAVE; }
    else if (vec == 2) { st = launch_tile<2, 2>(A, X, ldx, d, k0, Y, ldy, s); step = 4 * ISP_WAVE; }
    else if (w <= ISP_WAVE) { st = launch_tile<1, 1>(A, X, ldx, d, k0, Y, ldy, s); step = ISP_WAVE; }
    else if (w <= 2 * ISP_WAVE) { st = launch_tile<1, 2>(A, X, ldx, d, k0, Y, ldy, s); step = 2 * ISP_WAVE; }
    else { st = launch_tile<1, 4>(A, X, ldx, d, k0, Y, ldy, s); step = 4 * ISP_WAVE; }
    k0 += step;
  }
  return st;
}
