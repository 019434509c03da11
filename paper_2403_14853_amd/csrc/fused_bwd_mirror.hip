// Grouped FusedMM backward of a symmetric pattern in one pass, for 4 <= d <= 256 at any alignment.
#include "fused_grouped.h"

namespace {

// Backward in ONE pass over A when A^T's structure equals A's (symmetric pattern, ascending rows): entry p of
// row i names neighbour j, and position p of A^T holds the mirrored entry (j, i) with value a_ji.  Both sums of
// the backward then run over the same neighbours, and x_j and g_j are gathered once for both:
//   dX_i = sum_j (dz_ij + dz_ji) x_j + a_ji s g_j,   dz_ij = a_ij <g_i, x_j> f'(z),  dz_ji = a_ji <g_j, x_i> f'(z),
// z = <x_i, x_j> being the same for (i, j) and (j, i).  Two gathered rows per entry instead of three, one sweep
// over the index arrays instead of two.
struct g_args22 { const float* src[2]; int64_t lds_[2]; const float* rowop[2]; int64_t ldr[2]; float* out_entry; int op; const float* val2; };

template <int OP>
struct g_bwd_mirror {  // gathered x_j and g_j, row operands x_i and g_i
  static constexpr fused_pass PASS = fused_pass::one_pass;
  static constexpr int NSRC = 2, NROW = 2, RING4 = 4, RING8 = 2;
  static constexpr bool PER_ENTRY = false, ACCUMULATE = false, HAS_VAL2 = true;
  using args = g_args22;
  template <int LPG, int W, bool TAIL>
  __device__ static inline void edge(const args&, float a, float at, const float (&x)[2][W], const float (&r)[2][W],
                                     float (&acc)[W], const lane_cols<W / 4, TAIL>& lc) {
    float sg = 1.f, dsg = 0.f, gd_ij = 0.f, gd_ji = 0.f;
    if (OP != ISP_OP_ONE) {
      edge_fn(OP, group_allreduce<LPG>(dotw<W, TAIL>(r[0], x[0], lc)), sg, dsg);
      gd_ij = group_allreduce<LPG>(dotw<W, TAIL>(r[1], x[0], lc));  // <g_i, x_j>
      gd_ji = group_allreduce<LPG>(dotw<W, TAIL>(x[1], r[0], lc));  // <g_j, x_i>
    }
    const float w = at * sg;
    const float dz = (a * gd_ij + at * gd_ji) * dsg;
#pragma unroll
    for (int v = 0; v < W; ++v) acc[v] = fmaf(w, x[1][v], fmaf(dz, x[0][v], acc[v]));
  }
};

}  // namespace

isp_status isp_fused_grouped_bwd_mirror(const isp_csr* A, const float* X, int64_t ldx, const float* G, int64_t ldg, int d, int op, float* Y, int64_t ldy,
                              hipStream_t s) {
  g_args22 pa{{X, G}, {ldx, ldg}, {X, G}, {ldx, ldg}, nullptr, op, A->At->v.values};
  if (op == ISP_OP_SIGMOID) return run_grouped_d<g_bwd_mirror<ISP_OP_SIGMOID>>(A, pa, d, Y, ldy, s);
  if (op == ISP_OP_DOT) return run_grouped_d<g_bwd_mirror<ISP_OP_DOT>>(A, pa, d, Y, ldy, s);
  return run_grouped_d<g_bwd_mirror<ISP_OP_ONE>>(A, pa, d, Y, ldy, s);
}
