// SDDMM: out[p] = <U[i, :], V[col_p, :]> for every stored entry p of row i, in A's CSR order
// (paper Section 1: one of the two sparse operations GNN training rests on).  With U = dY and
// V = X this is the gradient of Y = A X with respect to A's stored values.
//
// Same work items as SpMM.  The wave keeps U's row in registers, gathers V's rows with the 64
// lanes spread over the feature dimension, and reduces each product across the wave.  Results
// of up to 64 consecutive entries are collected one per lane and stored coalesced.
#include "grouped_ops.h"
#include "lane_rule.h"

namespace {
using namespace isp_dev;

template <int VEC, bool HAS_VAL, bool SCALE, bool ADD>
__global__ void __launch_bounds__(ISP_WG) k_sddmm(isp_view A, const int64_t* __restrict__ indptr,
                                                  const int32_t* __restrict__ indices,
                                                  const float* __restrict__ values, const float* __restrict__ Um,
                                                  int64_t ldu, const float* __restrict__ Vm, int64_t ldv, int d, int k0,
                                                  float* __restrict__ out) {
  constexpr int U = 8;
  const int lane = threadIdx.x & (ISP_WAVE - 1);
  const int item = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * ISP_WAVES_PER_WG + (threadIdx.x >> 6)));
  if (item >= A.n_blocks + A.n_seg) return;
  const item_range it = locate_item(A, indptr, item);
  if (it.skip) return;
  const int col = k0 + lane * VEC;
  const bool on = col < d;

  int row = it.src_row;
  // segment items stay inside one row; block items walk rows [row, row_last)
  const int row_stop = it.is_seg ? row + 1 : it.row_last;
  int64_t p = it.p;
  const int64_t p_end = it.p_end;
  int64_t row_end = it.is_seg ? p_end : indptr[row + 1];
  while (row < row_stop && row_end == p && !it.is_seg) { ++row; row_end = (row < row_stop) ? indptr[row + 1] : INT64_MAX; }

  float u[VEC];
  auto load_u = [&]() {
#pragma unroll
    for (int v = 0; v < VEC; ++v) u[v] = 0.f;
    if (on && row < row_stop) load_vec<VEC>(Um + (int64_t)row * ldu + col, u);
  };
  load_u();

  while (p < p_end) {
    const int64_t left = p_end - p;
    const int cnt = left < ISP_WAVE ? (int)left : ISP_WAVE;
    int c = 0;
    float a = 1.f;
    if (lane < cnt) {
      c = __builtin_nontemporal_load(indices + p + lane);
      if (HAS_VAL && SCALE) a = __builtin_nontemporal_load(values + p + lane);
    }
    float res = 0.f;  // lane t ends up with the dot product of entry p + t
    for (int t = 0; t < cnt; t += U) {
      float x[U][VEC];
      const bool full = t + U <= cnt;
#pragma unroll
      for (int q = 0; q < U; ++q) {
        if (full || t + q < cnt) {
          const int cj = bcast_i(c, t + q);
#pragma unroll
          for (int v = 0; v < VEC; ++v) x[q][v] = 0.f;
          if (on) load_vec<VEC>(Vm + (int64_t)cj * ldv + col, x[q]);
        }
      }
#pragma unroll
      for (int q = 0; q < U; ++q) {
        if (full || t + q < cnt) {
          float part = 0.f;
#pragma unroll
          for (int v = 0; v < VEC; ++v) part = fmaf(u[v], x[q][v], part);
          const float dot = wave_allreduce(part);
          if (lane == t + q) res = dot;
          if (p + t + q + 1 == row_end && !it.is_seg) {
            ++row;
            row_end = (row < row_stop) ? indptr[row + 1] : INT64_MAX;
            while (row < row_stop && row_end == p + t + q + 1) { ++row; row_end = (row < row_stop) ? indptr[row + 1] : INT64_MAX; }
            load_u();
          }
        }
      }
    }
    if (lane < cnt) {
      if (HAS_VAL && SCALE) res *= a;
      if (ADD) res += out[p + lane];
      out[p + lane] = res;
    }
    p += cnt;
  }
}

// ---- grouped fast path (d >= 4, any alignment) ------------------------------------
// ADD: this pass covers a window of the feature columns and adds its partial dot product to out.
// The entry's staged value multiplies the dot product; it is 1 when the kernel is given no values
// (unscaled SDDMM, or a matrix without stored values).
template <bool ADD_ = false>
struct sddmm_policy {
  static constexpr int NSRC = 1, NROW = 1, RING4 = 4, RING8 = 4;
  static constexpr bool PER_ENTRY = true, ACCUMULATE = false, ADD = ADD_;
  struct args { const float* src[1]; int64_t lds_[1]; const float* rowop[1]; int64_t ldr[1]; float* out_entry; };
  template <int W, bool TAIL>
  __device__ static inline float partial(const float (&x)[1][W], const float (&r)[1][W], const lane_cols<W / 4, TAIL>& lc) {
    return dotw<W, TAIL>(r[0], x[0], lc);
  }
};

template <int LPG, int W, bool ADDR32, bool ADD, bool TAIL, int CAP>
__global__ void __launch_bounds__(ISP_WG) k_sddmm_grouped(isp_view A, const int64_t* __restrict__ indptr,
                                                          const int32_t* __restrict__ indices,
                                                          const float* __restrict__ values,
                                                          typename sddmm_policy<ADD>::args pa, int d, int k_lo) {
  __shared__ rn_lds_of<CAP> lds;
  fused_grouped_item<sddmm_policy<ADD>, LPG, W, ADDR32, TAIL>(A, indptr, indices, values, pa, d, nullptr, 0, lds, k_lo);
}

// One pass over the feature columns [k_lo, d_hi) (d_hi - k_lo <= W * LPG); add: accumulate into out.
template <int LPG, int W>
isp_status launch_grouped(const isp_csr* A, const float* U, int64_t ldu, const float* V, int64_t ldv, int k_lo,
                          int d_hi, bool add, bool scale, float* out, hipStream_t s) {
  const isp_view& v = A->v;
  const int n_items = v.n_blocks + v.n_seg;
  if (n_items == 0 || v.nnz == 0) return ISP_OK;
  const unsigned grid = (unsigned)((n_items + ISP_WAVES_PER_WG - 1) / ISP_WAVES_PER_WG);
  const float* vals = scale ? v.values : nullptr;
  const bool a32 = fused_offsets_fit_32(v.n_cols, ldv, d_hi) && fused_offsets_fit_32(v.n_rows, ldu, d_hi);
  const bool tail = (d_hi - k_lo) % 4 != 0;
#define ISP_GO(A32, AD, TL, CAP)                                                                                    \
  do {                                                                                                              \
    typename sddmm_policy<AD>::args pa{{V}, {ldv}, {U}, {ldu}, out};                                                 \
    k_sddmm_grouped<LPG, W, A32, AD, TL, CAP><<<grid, ISP_WG, 0, s>>>(v, v.indptr, v.indices, vals, pa, d_hi, k_lo);  \
  } while (0)
#define ISP_GO2(A32, AD, CAP) do { if (tail) ISP_GO(A32, AD, true, CAP); else ISP_GO(A32, AD, false, CAP); } while (0)
  if constexpr (LPG <= 16 && W == 4) {
    // Small tables only where the launch is long enough for the last workgroups to matter less: more than 12 per compute
    // unit, beyond 32 columns 15.  us with five / seven at a time: 13 k columns, 674 k entries: 24 columns 9.6 / 9.1; 39 k,
    // 993 k: 32 13.7 / 12.5, but 56 21.7 / 21.8; 111 k, 1.4 M: 40 29.1 / 30.1; 43 k, 1.2 M: 32 17.9 / 16.0; 42 k, 1.5 M: 48 29.2 /
    // 26.7; 35 k, 870 k: 54 19.6 / 20.0; 51 k, 1 M: 8 12.4 / 12.1; 100 k, 1 M: 32 14.2 / 13.3, 64 21.5 / 22.3.  Never beyond 64 columns, where they made
    // little difference either way (10 k, 1 M: 128 30.4 / 29.4).
    if (a32 && rn_small_tables(A, v, d_hi - k_lo, grid, d_hi - k_lo <= 32 ? 12 : 15)) {
      if (add) ISP_GO2(true, true, RN_SMALL); else ISP_GO2(true, false, RN_SMALL);
      ISP_LAUNCH_CHECK();
      return ISP_OK;
    }
  }
  if (a32) { if (add) ISP_GO2(true, true, GS_MAX_ENT); else ISP_GO2(true, false, GS_MAX_ENT); }
  else { if (add) ISP_GO2(false, true, GS_MAX_ENT); else ISP_GO2(false, false, GS_MAX_ENT); }
#undef ISP_GO2
#undef ISP_GO
  ISP_LAUNCH_CHECK();
  return ISP_OK;
}

template <int VEC>
isp_status launch(const isp_csr* A, const float* U, int64_t ldu, const float* V, int64_t ldv, int d, int k0,
                  bool scale, bool add, float* out, hipStream_t s) {
  const isp_view& v = A->v;
  const int n_items = v.n_blocks + v.n_seg;
  if (n_items == 0 || v.nnz == 0) return ISP_OK;
  const unsigned grid = (unsigned)((n_items + ISP_WAVES_PER_WG - 1) / ISP_WAVES_PER_WG);
  const bool sc = scale && v.values;
#define ISP_SDDMM_GO(HV, SC, AD) \
  k_sddmm<VEC, HV, SC, AD><<<grid, ISP_WG, 0, s>>>(v, v.indptr, v.indices, v.values, U, ldu, V, ldv, d, k0, out)
  if (sc) { if (add) ISP_SDDMM_GO(true, true, true); else ISP_SDDMM_GO(true, true, false); }
  else { if (add) ISP_SDDMM_GO(false, false, true); else ISP_SDDMM_GO(false, false, false); }
#undef ISP_SDDMM_GO
  ISP_LAUNCH_CHECK();
  return ISP_OK;
}

// Below this size rows wider than 256 columns go 512 at a time (64 lanes, two float4): a pass there is the time of its chains, and two
// passes stage every entry twice (us, 256 / 512 at a time: R-MAT, 1.5 k rows, 8 k entries, 344 columns 11.8 / 8.6; 4 k, 17 k, 432: 14.2 / 10.4; 20 k,
// 79 k, 344: 21.7 / 18.0; 10 k, 204 k, 368: 33.5 / 29.8; 13 k, 445 k, 376: 54.8 / 51.0; uniform, 21 k, 420 k, 544: 124 / 125; but 111 k, 801 k, 584: 235 / 247;
// 11 k, 1.1 M, 272: 130 / 156; 58 k, 1.9 M, 336: 191 / 197).
constexpr int64_t SDDMM_WIDE_NNZ = 3 << 18;

constexpr int64_t SLICE_FLOATS = 16 << 20;  // V of 64 MB, twice the L2s

bool aligned(const void* p, size_t a) { return ((uintptr_t)p & (a - 1)) == 0; }

}  // namespace

isp_status isp_sddmm_launch(const isp_csr* A, const float* U, int64_t ldu, const float* V, int64_t ldv, int32_t d,
                            bool scale, float* out, hipStream_t s) {
  const isp_view& av = A->v;
  const bool grouped_ok = d >= 4 && A->info.block_cost <= GS_MAX_ROWS &&
                          A->info.block_cost + av.hub_t <= GS_MAX_ENT && av.seg_len <= GS_MAX_ENT &&
                          !A->tune.no_grouped;
  if (grouped_ok) {
    // One pass covers a window of the feature columns; later passes add their partial dot products.
    //  - big graphs with many columns, rows of whole 64-float halves: 64-column passes, so that every L2 holds
    //    half-rows of twice as many hot columns (the same effect, under the same conditions, as the column
    //    slices of SpMM);
    //  - otherwise rows wider than 128 floats go 128 columns at a time on the big graphs, and on others whose V is
    //    beyond the L2s, where that cuts no cache line (us in one pass -> in windows, 2.4 M / 3 M entries: 256 columns 219 -> 189 / 307 -> 281, 192
    //    161 -> 143 / 228 -> 203; at 200 columns it would be 187 -> 210 / 261 -> 299), 256 on the rest.  (On big graphs windows were the better way for
    //    whole lines; for ragged rows they need not be: 248 columns, 1 M columns, 16.9 M entries 1877 in one pass, 2087 in windows.)
    const bool big = av.nnz >= ((int64_t)8 << 20);
    int wp = d;
    if (big && av.n_cols >= (1 << 19) && d > ISP_WAVE && d % ISP_WAVE == 0 && ldu % 32 == 0 && ldv % 32 == 0 &&
        !A->tune.sddmm_one_pass)
      wp = ISP_WAVE;
    else if (d > 2 * ISP_WAVE && (big || (ldu % 32 == 0 && ldv % 32 == 0 && av.n_cols * ldv >= SLICE_FLOATS))) wp = 2 * ISP_WAVE;
    else if (d > ISP_PARTIAL_TILE) wp = av.nnz < SDDMM_WIDE_NNZ ? 2 * ISP_PARTIAL_TILE : ISP_PARTIAL_TILE;
    isp_status st = ISP_OK;
    for (int k_lo = 0, k_next; k_lo < d && st == ISP_OK; k_lo = k_next) {
      int k_hi = k_lo + wp < d ? k_lo + wp : d;
      if (k_hi < d && d - k_hi < 4) k_hi = d - 4;  // (no window narrower than a float4 lane)
      const int w = k_hi - k_lo;
      const bool add = k_lo > 0;
      k_next = k_hi;
      // One float4 per lane up to 128 columns (two, which serve twice the entries per step, load the row operand with
      // every step and hold twice the registers: 128 columns in one pass, us, one / two: 115 M entries 2558 / 2702, 2.4 M 93 / 98,
      // 1.2 M 48.9 / 50.0), two above: with one, a wavefront has a single run.  That is only the better way for nearly full rows on graphs
      // with work for several times as many wavefronts as the chip holds (248 columns, us, one / two: 108 k entries
      // 21.8 / 16.8, 1.2 M 116 / 119, 2.4 M 236 / 249, 3 M 325 / 342; 160 columns: 108 k 21.3 / 15.0, 589 k 42.2 / 39.4, 1.2 M 83.8 / 74.1).  In between, one is the better
      // way already at 589 k entries from 200 columns (45.1 / 47.8, 248 columns 51.7 / 57.5).  On small matrices, where a wavefront's run is what the
      // launch takes, two are the better way from 65 columns up (R-MAT, 2.4 k rows, 46 k entries, 104 columns 6.9 / 5.6; 2.8 k, 64 k, 122: 6.8 / 5.6; 7 k, 186 k,
      // 88: 10.2 / 9.2; 13 k, 247 k, 70: 13.0 / 11.3; uniform, 4.9 k, 67 k, 96: 6.5 / 5.9; but 31 k, 374 k, 120: 28.0 / 29.7).
      if (sddmm_four_lanes(w, av.nnz, av.n_hub)) st = launch_grouped<4, 4>(A, U, ldu, V, ldv, k_lo, k_hi, add, scale, out, s);
      else if (w <= 32) st = launch_grouped<8, 4>(A, U, ldu, V, ldv, k_lo, k_hi, add, scale, out, s);
      else if (w <= 64) st = launch_grouped<16, 4>(A, U, ldu, V, ldv, k_lo, k_hi, add, scale, out, s);
      else if (w <= 128 && av.nnz < (1 << 18)) st = launch_grouped<16, 8>(A, U, ldu, V, ldv, k_lo, k_hi, add, scale, out, s);
      else if (w <= 128) st = launch_grouped<32, 4>(A, U, ldu, V, ldv, k_lo, k_hi, add, scale, out, s);
      else if (w > ISP_PARTIAL_TILE) st = launch_grouped<64, 8>(A, U, ldu, V, ldv, k_lo, k_hi, add, scale, out, s);
      else if (w <= 192 || av.nnz < (1 << 20)) st = launch_grouped<32, 8>(A, U, ldu, V, ldv, k_lo, k_hi, add, scale, out, s);
      else st = launch_grouped<64, 4>(A, U, ldu, V, ldv, k_lo, k_hi, add, scale, out, s);
    }
    return st;
  }
  int vec = 1;
  if (d > 2 * ISP_WAVE && d % 4 == 0 && ldu % 4 == 0 && ldv % 4 == 0 && aligned(U, 16) && aligned(V, 16)) vec = 4;
  else if (d > ISP_WAVE && d % 2 == 0 && ldu % 2 == 0 && ldv % 2 == 0 && aligned(U, 8) && aligned(V, 8)) vec = 2;
  isp_status st = ISP_OK;
  // feature tiles of 64 * vec columns; the first tile writes out, later tiles add their partial dot products
  for (int k0 = 0; k0 < d && st == ISP_OK; k0 += ISP_WAVE * vec) {
    const bool add = k0 > 0;
    if (vec == 4) st = launch<4>(A, U, ldu, V, ldv, d, k0, scale, add, out, s);
    else if (vec == 2) st = launch<2>(A, U, ldu, V, ldv, d, k0, scale, add, out, s);
    else st = launch<1>(A, U, ldu, V, ldv, d, k0, scale, add, out, s);
  }
  return st;
}
