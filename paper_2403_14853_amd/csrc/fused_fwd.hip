// Grouped FusedMM forward: y_i = sum_p a_p s_p x_j, s_p = f(<x_i, x_j>), for 4 <= d <= 256 at any alignment.
#include "fused_grouped.h"

namespace {

struct g_args1 { const float* src[1]; int64_t lds_[1]; const float* rowop[1]; int64_t ldr[1]; float* out_entry; int op; };

template <int OP>
struct g_fwd {  // gathered x_j, row operand x_i
  static constexpr int NSRC = 1, NROW = 1, RING4 = 4, RING8 = 4;
  static constexpr bool PER_ENTRY = false, ACCUMULATE = false;
  using args = g_args1;
  template <int LPG, int W, bool TAIL>
  __device__ static inline void edge(const args&, float a, const float (&x)[1][W], const float (&r)[1][W],
                                     float (&acc)[W], const lane_cols<W / 4, TAIL>& lc) {
    float sg = 1.f, dsg = 0.f;
    if (OP != ISP_OP_ONE) edge_fn(OP, group_allreduce<LPG>(dotw<W, TAIL>(r[0], x[0], lc)), sg, dsg);
    const float w = a * sg;
#pragma unroll
    for (int v = 0; v < W; ++v) acc[v] = fmaf(w, x[0][v], acc[v]);
  }
};

}  // namespace

isp_status isp_fused_grouped_fwd(const isp_csr* A, const float* X, int64_t ldx, int d, int op, float* Y, int64_t ldy, hipStream_t s) {
  g_args1 pa{{X}, {ldx}, {X}, {ldx}, nullptr, op};
  if (op == ISP_OP_SIGMOID) return run_grouped_d<g_fwd<ISP_OP_SIGMOID>>(A, pa, d, Y, ldy, s);
  if (op == ISP_OP_DOT) return run_grouped_d<g_fwd<ISP_OP_DOT>>(A, pa, d, Y, ldy, s);
  return run_grouped_d<g_fwd<ISP_OP_ONE>>(A, pa, d, Y, ldy, s);
}
