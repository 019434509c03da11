// Grouped FusedMM backward, row pass over A^T: dX_j += sum_p (a_p s_p g_i + dz_p x_i), for 4 <= d <= 256 at any
// alignment.  A is the transpose's handle here.
#include "fused_grouped.h"

namespace {

struct g_args21 { const float* src[2]; int64_t lds_[2]; const float* rowop[1]; int64_t ldr[1]; float* out_entry; int op; };

template <int OP>
struct g_bwd_col {  // over A^T: gathered x_i and g_i, row operand x_j:  dX_j += a s g_i + dz x_i
  static constexpr fused_pass PASS = fused_pass::two_pass;
  static constexpr int NSRC = 2, NROW = 1, RING4 = 4, RING8 = 2;
  static constexpr bool PER_ENTRY = false, ACCUMULATE = true;
  // (two entries at a time: figures with the row pass's policy; the one-pass backward of symmetric patterns, with three dot products and twice the
  // registers, gains nothing: 149.2 / 149.6, 326 / 327, 80.4 / 80.2)
  static constexpr int NDOT = OP != ISP_OP_ONE ? 2 : 0, NSCAL = 2, PAIR_LPG = 16;
  using args = g_args21;
  template <int W, bool TAIL>
  __device__ static inline void dots(const float (&x)[2][W], const float (&r)[1][W], const lane_cols<W / 4, TAIL>& lc, float* p) {
    p[0] = dotw<W, TAIL>(r[0], x[0], lc);
    p[1] = dotw<W, TAIL>(r[0], x[1], lc);
  }
  __device__ static inline void scalars(const float* t, float* s) {
    float dsg;
    edge_fn(OP, t[0], s[0], dsg);
    s[1] = t[1] * dsg;
  }
  template <int W>
  __device__ static inline void apply(float a, const float* s, const float (&x)[2][W], float (&acc)[W]) {
    const float w = a * s[0], dz = a * s[1];
#pragma unroll
    for (int v = 0; v < W; ++v) acc[v] = fmaf(w, x[1][v], fmaf(dz, x[0][v], acc[v]));
  }
};

}  // namespace

isp_status isp_fused_grouped_bwd_col(const isp_csr* A, const float* X, int64_t ldx, const float* G, int64_t ldg, int d, int op, float* Y, int64_t ldy,
                              hipStream_t s) {
  g_args21 pa{{X, G}, {ldx, ldg}, {X}, {ldx}, nullptr, op};
  if (op == ISP_OP_SIGMOID) return run_grouped_d<g_bwd_col<ISP_OP_SIGMOID>>(A, pa, d, Y, ldy, s);
  if (op == ISP_OP_DOT) return run_grouped_d<g_bwd_col<ISP_OP_DOT>>(A, pa, d, Y, ldy, s);
  return run_grouped_d<g_bwd_col<ISP_OP_ONE>>(A, pa, d, Y, ldy, s);
}
