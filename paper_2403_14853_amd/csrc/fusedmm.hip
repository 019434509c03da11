// FusedMM, sigmoid instance (paper Section 1(a): SDDMM and SpMM combined into one operation):
//   forward   s_p = sigmoid(<x_i, x_j>),  y_i = sum_p a_p s_p x_j            (j = column of p)
//   backward  dz_p = a_p <g_i, x_j> s_p (1 - s_p)
//             dX_i = sum_{p in row i} dz_p x_j + sum_{p in column i} (a_p s_p g_r + dz_p x_r)
// The per-edge scores exist only in registers: each gathered row x_j is used for the dot product
// and for the accumulation in the same pass, and the backward recomputes the scores instead of
// reading them back.  The column sum of the backward runs over the rows of the cached transpose.
#include "fused_grouped.h"

namespace {
using namespace isp_dev;

template <int VEC, int T>
__device__ inline float dot_lanes(const float (&a)[T][VEC], const float (&b)[T][VEC]) {
  float s = 0.f;
#pragma unroll
  for (int tt = 0; tt < T; ++tt)
#pragma unroll
    for (int v = 0; v < VEC; ++v) s = fmaf(a[tt][v], b[tt][v], s);
  return s;
}

template <int VEC, int T>
__device__ inline void load_row(const float* __restrict__ M, int64_t ld, int row, const int (&col)[T],
                                const bool (&on)[T], float (&o)[T][VEC]) {
#pragma unroll
  for (int tt = 0; tt < T; ++tt) {
#pragma unroll
    for (int v = 0; v < VEC; ++v) o[tt][v] = 0.f;
    if (on[tt]) load_vec<VEC>(M + (int64_t)row * ld + col[tt], o[tt]);
  }
}

constexpr int pick_u(int regs_per_edge) { return regs_per_edge >= 8 ? 2 : (regs_per_edge >= 4 ? 4 : 8); }

// ---- forward ---------------------------------------------------------------------------------
template <int VEC_, int T_, bool HAS_VAL_>
struct fwd_policy {
  static constexpr int VEC = VEC_, T = T_, NG = 1, U = pick_u(VEC_ * T_);
  static constexpr bool HAS_VAL = HAS_VAL_, ACCUMULATE = false, NEEDS_PERM = false, HAS_FINISH = false;
  struct args { const float* src[1]; int64_t ld[1]; int op; };
  struct row_state { float xi[T][VEC]; };
  __device__ static inline void row_begin(const args& pa, row_state& rs, int row, const int (&col)[T],
                                          const bool (&on)[T]) {
    load_row<VEC, T>(pa.src[0], pa.ld[0], row, col, on, rs.xi);
  }
  __device__ static inline void edge(const args& pa, row_state& rs, float a, const float (&x)[1][T][VEC],
                                     float (&acc)[T][VEC], const bool (&)[T], const edge_info&) {
    float sg = 1.f, dsg = 0.f;
    if (pa.op != ISP_OP_ONE) edge_fn(pa.op, wave_allreduce(dot_lanes<VEC, T>(rs.xi, x[0])), sg, dsg);
    const float w = a * sg;
#pragma unroll
    for (int tt = 0; tt < T; ++tt)
#pragma unroll
      for (int v = 0; v < VEC; ++v) acc[tt][v] = fmaf(w, x[0][tt][v], acc[tt][v]);
  }
};

// ---- backward, row pass over A: dX_i = sum_p dz_p x_j ----------------------------------------
template <int VEC_, int T_, bool HAS_VAL_>
struct bwd_row_policy {
  static constexpr int VEC = VEC_, T = T_, NG = 1, U = pick_u(VEC_ * T_);
  static constexpr bool HAS_VAL = HAS_VAL_, ACCUMULATE = false, NEEDS_PERM = false, HAS_FINISH = false;
  struct args { const float* src[1]; int64_t ld[1]; const float* G; int64_t ldg; int op; };
  struct row_state { float xi[T][VEC]; float gi[T][VEC]; };
  __device__ static inline void row_begin(const args& pa, row_state& rs, int row, const int (&col)[T],
                                          const bool (&on)[T]) {
    load_row<VEC, T>(pa.src[0], pa.ld[0], row, col, on, rs.xi);
    load_row<VEC, T>(pa.G, pa.ldg, row, col, on, rs.gi);
  }
  __device__ static inline void edge(const args& pa, row_state& rs, float a, const float (&x)[1][T][VEC],
                                     float (&acc)[T][VEC], const bool (&)[T], const edge_info&) {
    if (pa.op == ISP_OP_ONE) return;  // s does not depend on x_i: nothing flows through z
    const float z = wave_allreduce(dot_lanes<VEC, T>(rs.xi, x[0]));
    const float gd = wave_allreduce(dot_lanes<VEC, T>(rs.gi, x[0]));
    float sg, dsg;
    edge_fn(pa.op, z, sg, dsg);
    const float dz = a * gd * dsg;
#pragma unroll
    for (int tt = 0; tt < T; ++tt)
#pragma unroll
      for (int v = 0; v < VEC; ++v) acc[tt][v] = fmaf(dz, x[0][tt][v], acc[tt][v]);
  }
};

// ---- backward, row pass over A^T: dX_j += sum_p (a_p s_p g_i + dz_p x_i) ---------------------
// Row j of A^T lists the source rows i of the entries in column j; x_i and g_i are gathered.
template <int VEC_, int T_, bool HAS_VAL_>
struct bwd_col_policy {
  static constexpr int VEC = VEC_, T = T_, NG = 2, U = pick_u(2 * VEC_ * T_);
  static constexpr bool HAS_VAL = HAS_VAL_, ACCUMULATE = true, NEEDS_PERM = false, HAS_FINISH = false;
  struct args { const float* src[2]; int64_t ld[2]; int op; };  // src[0] = X, src[1] = dY
  struct row_state { float xj[T][VEC]; };
  __device__ static inline void row_begin(const args& pa, row_state& rs, int row, const int (&col)[T],
                                          const bool (&on)[T]) {
    load_row<VEC, T>(pa.src[0], pa.ld[0], row, col, on, rs.xj);
  }
  __device__ static inline void edge(const args& pa, row_state& rs, float a, const float (&x)[2][T][VEC],
                                     float (&acc)[T][VEC], const bool (&)[T], const edge_info&) {
    float sg = 1.f, dsg = 0.f, gd = 0.f;
    if (pa.op != ISP_OP_ONE) {
      edge_fn(pa.op, wave_allreduce(dot_lanes<VEC, T>(rs.xj, x[0])), sg, dsg);
      gd = wave_allreduce(dot_lanes<VEC, T>(rs.xj, x[1]));
    }
    const float w = a * sg;
    const float dz = a * gd * dsg;
#pragma unroll
    for (int tt = 0; tt < T; ++tt)
#pragma unroll
      for (int v = 0; v < VEC; ++v) acc[tt][v] = fmaf(w, x[1][tt][v], fmaf(dz, x[0][tt][v], acc[tt][v]));
  }
};

template <class P>
__global__ void __launch_bounds__(ISP_WG) k_fused(isp_view A, const int64_t* __restrict__ indptr,
                                                  const int32_t* __restrict__ indices,
                                                  const float* __restrict__ values, typename P::args pa, int d,
                                                  float* __restrict__ Y, int64_t ldy, int store_group, int group_cnt) {
  stream_item<P>(A, indptr, indices, values, pa, d, 0, Y, ldy, store_group, group_cnt);
}

template <int VEC, bool ACC>
__global__ void __launch_bounds__(ISP_WG) k_fused_fixup_group(isp_view A, int d, int k0, float* __restrict__ Y,
                                                              int64_t ldy, int stride, int slot) {
  hub_fixup<VEC, 1, ACC>(A, d, k0, Y, ldy, stride, slot);
}

// store_group < 0: one launch covers all d <= 256 columns.  Otherwise (wider rows) hub segments compute with
// whole rows and store column groups [store_group, store_group + group_cnt), one partial row per group, and
// one fix-up per group adds them; the row blocks do all their work in the launch that starts at group 0.
template <class P>
isp_status run_pass(const isp_csr* A, const typename P::args& pa, int d, float* Y, int64_t ldy, hipStream_t s,
                    int store_group = -1, int group_cnt = 1) {
  const isp_view& v = A->v;
  const int n_items = v.n_blocks + v.n_seg;
  if (n_items > 0) {
    const unsigned grid = (unsigned)((n_items + ISP_WAVES_PER_WG - 1) / ISP_WAVES_PER_WG);
    k_fused<P><<<grid, ISP_WG, 0, s>>>(v, v.indptr, v.indices, v.values, pa, d, Y, ldy, store_group, group_cnt);
    ISP_LAUNCH_CHECK();
  }
  if (v.n_hub > 0) {
    const unsigned grid = (unsigned)((v.n_hub + ISP_WAVES_PER_WG - 1) / ISP_WAVES_PER_WG);
    if (store_group < 0) {
      k_fused_fixup<P::VEC, P::T, P::ACCUMULATE><<<grid, ISP_WG, 0, s>>>(v, d, Y, ldy);
      ISP_LAUNCH_CHECK();
    } else {
      for (int g = 0; g < group_cnt; ++g) {
        k_fused_fixup_group<P::VEC, P::ACCUMULATE><<<grid, ISP_WG, 0, s>>>(v, d, (store_group + g) * ISP_WAVE * P::VEC, Y,
                                                                          ldy, group_cnt, g);
        ISP_LAUNCH_CHECK();
      }
    }
  }
  return ISP_OK;
}

// Column groups (of 256) a hub segment may store per launch of a wide pass: as many as the partial-row scratch
// holds for all segments at once (the scratch is sized for the worst-case segment count, usually several times
// the actual one), at least one.  ISP_WIDE_GROUPS (read at build) caps it, for tests.
int groups_per_launch(const isp_csr* A, int n_groups) {
  int64_t gc = A->v.n_seg > 0 ? A->partial_rows / A->v.n_seg : n_groups;
  if (A->tune.wide_groups > 0 && gc > A->tune.wide_groups) gc = A->tune.wide_groups;
  return gc < 1 ? 1 : (gc > n_groups ? n_groups : (int)gc);
}

bool grouped_partition_ok(const isp_csr* A) {
  return A->info.block_cost <= GS_MAX_ROWS && A->info.block_cost + A->v.hub_t <= GS_MAX_ENT &&
         A->v.seg_len <= GS_MAX_ENT && !A->tune.no_grouped;
}

bool aligned(const void* p, size_t a) { return ((uintptr_t)p & (a - 1)) == 0; }

// 0: float4 lanes, 1: float2 lanes, 2..4: scalar lanes with 1, 2, 4 column groups
int pick_shape(int d, bool ok4, bool ok2) {
  if (d > 2 * ISP_WAVE && d % 4 == 0 && ok4) return 0;
  if (d > ISP_WAVE && d <= 2 * ISP_WAVE && d % 2 == 0 && ok2) return 1;
  if (d <= ISP_WAVE) return 2;
  if (d <= 2 * ISP_WAVE) return 3;
  return 4;
}

#define ISP_SHAPE_SWITCH(shape, has_val, CALL)                                   \
  switch (shape) {                                                              \
    case 0: if (has_val) { CALL(4, 1, true); } else { CALL(4, 1, false); } break; \
    case 1: if (has_val) { CALL(2, 1, true); } else { CALL(2, 1, false); } break; \
    case 2: if (has_val) { CALL(1, 1, true); } else { CALL(1, 1, false); } break; \
    case 3: if (has_val) { CALL(1, 2, true); } else { CALL(1, 2, false); } break; \
    default: if (has_val) { CALL(1, 4, true); } else { CALL(1, 4, false); } break; \
  }

}  // namespace

isp_status isp_fusedmm_launch(const isp_csr* A, const float* X, int64_t ldx, int32_t d, int op, float* Y,
                              int64_t ldy, hipStream_t s) {
  const bool ok4 = ldx % 4 == 0 && ldy % 4 == 0 && aligned(X, 16) && aligned(Y, 16);
  const bool ok2 = ldx % 2 == 0 && ldy % 2 == 0 && aligned(X, 8) && aligned(Y, 8);
  if (d >= 4 && d <= ISP_PARTIAL_TILE && grouped_partition_ok(A)) {
    return isp_fused_grouped_fwd(A, X, ldx, d, op, Y, ldy, s);
  }
  const bool hv = A->v.values != nullptr;
  isp_status st = ISP_OK;
  if (d > ISP_PARTIAL_TILE) {
    // wider than a hub partial row: whole rows in the arithmetic (the score needs them), 256 columns stored
    // per launch (the caller has checked d <= 1024)
    if (!(ok4 && d % 4 == 0))
      return isp_fail(ISP_EUNSUPPORTED, "FusedMM with d > %d needs d %% 4 == 0 and 16-byte aligned rows", ISP_PARTIAL_TILE);
    const int n_groups = (d + ISP_PARTIAL_TILE - 1) / ISP_PARTIAL_TILE;
    const int gc = groups_per_launch(A, n_groups);
    for (int w = 0; w < n_groups && st == ISP_OK; w += gc) {
      const int cnt = n_groups - w < gc ? n_groups - w : gc;
#define ISP_WIDE(T, HV)                             \
  {                                                 \
    using P = fwd_policy<4, T, HV>;                 \
    P::args pa;                                     \
    pa.src[0] = X;                                  \
    pa.ld[0] = ldx;                                 \
    pa.op = op;                                     \
    st = run_pass<P>(A, pa, d, Y, ldy, s, w, cnt);  \
  }
      if (n_groups <= 2) { if (hv) ISP_WIDE(2, true) else ISP_WIDE(2, false) }
      else { if (hv) ISP_WIDE(4, true) else ISP_WIDE(4, false) }
#undef ISP_WIDE
    }
    return st;
  }
  const int shape = pick_shape(d, ok4, ok2);
#define ISP_FWD(V, T, HV)                         \
  {                                               \
    using P = fwd_policy<V, T, HV>;               \
    P::args pa;                                   \
    pa.src[0] = X;                                \
    pa.ld[0] = ldx;                               \
    pa.op = op;                                   \
    st = run_pass<P>(A, pa, d, Y, ldy, s);        \
  }
  ISP_SHAPE_SWITCH(shape, hv, ISP_FWD)
#undef ISP_FWD
  return st;
}

isp_status isp_fusedmm_bwd_launch(const isp_csr* A, const float* X, int64_t ldx, const float* G, int64_t ldg,
                                  int32_t d, int op, float* dX, int64_t lddx, hipStream_t s) {
  const bool ok4 = ldx % 4 == 0 && ldg % 4 == 0 && lddx % 4 == 0 && aligned(X, 16) && aligned(G, 16) && aligned(dX, 16);
  const bool ok2 = ldx % 2 == 0 && ldg % 2 == 0 && lddx % 2 == 0 && aligned(X, 8) && aligned(G, 8) && aligned(dX, 8);
  if (d >= 4 && d <= ISP_PARTIAL_TILE && grouped_partition_ok(A) && A->mirror_aligned && !A->tune.no_mirror) {
    // symmetric pattern: one pass over A serves both sums (the mirrored entries' values are A^T's)
    return isp_fused_grouped_bwd_mirror(A, X, ldx, G, ldg, d, op, dX, lddx, s);
  }
  if (d >= 4 && d <= ISP_PARTIAL_TILE && grouped_partition_ok(A) && grouped_partition_ok(A->At)) {
    const isp_status st1 = isp_fused_grouped_bwd_row(A, X, ldx, G, ldg, d, op, dX, lddx, s);
    return st1 != ISP_OK ? st1 : isp_fused_grouped_bwd_col(A->At, X, ldx, G, ldg, d, op, dX, lddx, s);
  }
  const bool hv = A->v.values != nullptr;
  isp_status st = ISP_OK;
  if (d > ISP_PARTIAL_TILE) {  // as in the forward: whole rows in the arithmetic, one column group stored per launch
    if (!(ok4 && d % 4 == 0))
      return isp_fail(ISP_EUNSUPPORTED, "FusedMM with d > %d needs d %% 4 == 0 and 16-byte aligned rows", ISP_PARTIAL_TILE);
    const int n_groups = (d + ISP_PARTIAL_TILE - 1) / ISP_PARTIAL_TILE;
    // every row pass before the first column pass: the column pass of group 0 already adds to all columns of
    // the rows that are not hubs of A^T, which a later row pass's fix-up must not overwrite
#define ISP_WIDE_ROW(T, HV)                                              \
  {                                                                      \
    using P1 = bwd_row_policy<4, T, HV>;                                 \
    P1::args p1;                                                         \
    p1.src[0] = X; p1.ld[0] = ldx; p1.G = G; p1.ldg = ldg; p1.op = op;   \
    st = run_pass<P1>(A, p1, d, dX, lddx, s, w, cnt);                    \
  }
#define ISP_WIDE_COL(T, HV)                                              \
  {                                                                      \
    using P2 = bwd_col_policy<4, T, HV>;                                 \
    P2::args p2;                                                         \
    p2.src[0] = X; p2.ld[0] = ldx; p2.src[1] = G; p2.ld[1] = ldg; p2.op = op; \
    st = run_pass<P2>(A->At, p2, d, dX, lddx, s, w, cnt);                \
  }
    const int gc1 = groups_per_launch(A, n_groups), gc2 = groups_per_launch(A->At, n_groups);
    for (int w = 0; w < n_groups && st == ISP_OK; w += gc1) {
      const int cnt = n_groups - w < gc1 ? n_groups - w : gc1;
      if (n_groups <= 2) { if (hv) ISP_WIDE_ROW(2, true) else ISP_WIDE_ROW(2, false) }
      else { if (hv) ISP_WIDE_ROW(4, true) else ISP_WIDE_ROW(4, false) }
    }
    for (int w = 0; w < n_groups && st == ISP_OK; w += gc2) {
      const int cnt = n_groups - w < gc2 ? n_groups - w : gc2;
      if (n_groups <= 2) { if (hv) ISP_WIDE_COL(2, true) else ISP_WIDE_COL(2, false) }
      else { if (hv) ISP_WIDE_COL(4, true) else ISP_WIDE_COL(4, false) }
    }
#undef ISP_WIDE_ROW
#undef ISP_WIDE_COL
    return st;
  }
  const int shape = pick_shape(d, ok4, ok2);
#define ISP_BWD(V, T, HV)                                  \
  {                                                        \
    using P1 = bwd_row_policy<V, T, HV>;                   \
    P1::args p1;                                           \
    p1.src[0] = X; p1.ld[0] = ldx; p1.G = G; p1.ldg = ldg; p1.op = op; \
    st = run_pass<P1>(A, p1, d, dX, lddx, s);              \
    if (st == ISP_OK) {                                    \
      using P2 = bwd_col_policy<V, T, HV>;                 \
      P2::args p2;                                         \
      p2.src[0] = X; p2.ld[0] = ldx; p2.src[1] = G; p2.ld[1] = ldg; p2.op = op; \
      st = run_pass<P2>(A->At, p2, d, dX, lddx, s);        \
    }                                                      \
  }
  ISP_SHAPE_SWITCH(shape, hv, ISP_BWD)
#undef ISP_BWD
  return st;
}
