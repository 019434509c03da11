// Grouped FusedMM backward, row pass over A: dX_i = sum_p dz_p x_j, for 4 <= d <= 256 at any alignment.
#include "fused_grouped.h"

namespace {

struct g_args12 { const float* src[1]; int64_t lds_[1]; const float* rowop[2]; int64_t ldr[2]; float* out_entry; int op; };

template <int OP>
struct g_bwd_row {  // gathered x_j, row operands x_i and g_i:  dX_i += dz x_j
  static constexpr fused_pass PASS = fused_pass::two_pass;
  static constexpr int NSRC = 1, NROW = 2, RING4 = 4, RING8 = 2;
  static constexpr bool PER_ENTRY = false, ACCUMULATE = false;
  // Two entries at a time, us of the whole backward of a directed graph (both passes) one / two: R-MAT, 60 k rows, 1.5 M entries: 64 columns 105.6 / 102,
  // 128 194 / 181, 256 433 / 405; 200 k, 4 M: 264 / 259, 584 / 560, 1414 / 1401; 1 M, 17 M: 1277 / 1264, 128 2883 / 2850; with 8 lanes, 32 columns,
  // 607 / 607.
  static constexpr int NDOT = OP != ISP_OP_ONE ? 2 : 0, NSCAL = 1, PAIR_LPG = 16;
  using args = g_args12;
  template <int W, bool TAIL>
  __device__ static inline void dots(const float (&x)[1][W], const float (&r)[2][W], const lane_cols<W / 4, TAIL>& lc, float* p) {
    p[0] = dotw<W, TAIL>(r[0], x[0], lc);
    p[1] = dotw<W, TAIL>(r[1], x[0], lc);
  }
  __device__ static inline void scalars(const float* t, float* s) {
    float sg, dsg;
    edge_fn(OP, t[0], sg, dsg);
    s[0] = t[1] * dsg;
  }
  template <int W>
  __device__ static inline void apply(float a, const float* s, const float (&x)[1][W], float (&acc)[W]) {
    if (OP == ISP_OP_ONE) return;  // s does not depend on x_i: nothing flows through z
    const float dz = a * s[0];
#pragma unroll
    for (int v = 0; v < W; ++v) acc[v] = fmaf(dz, x[0][v], acc[v]);
  }
};

}  // namespace

isp_status isp_fused_grouped_bwd_row(const isp_csr* A, const float* X, int64_t ldx, const float* G, int64_t ldg, int d, int op, float* Y, int64_t ldy,
                              hipStream_t s) {
  g_args12 pa{{X}, {ldx}, {X, G}, {ldx, ldg}, nullptr, op};
  if (op == ISP_OP_SIGMOID) return run_grouped_d<g_bwd_row<ISP_OP_SIGMOID>>(A, pa, d, Y, ldy, s);
  if (op == ISP_OP_DOT) return run_grouped_d<g_bwd_row<ISP_OP_DOT>>(A, pa, d, Y, ldy, s);
  return run_grouped_d<g_bwd_row<ISP_OP_ONE>>(A, pa, d, Y, ldy, s);
}
