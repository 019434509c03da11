// Grouped FusedMM forward: y_i = sum_p a_p s_p x_j, s_p = f(<x_i, x_j>), for 4 <= d <= 256 at any alignment.
#include "fused_grouped.h"

namespace {

struct g_args1 { const float* src[1]; int64_t lds_[1]; const float* rowop[1]; int64_t ldr[1]; float* out_entry; int op; };

template <int OP>
struct g_fwd {  // gathered x_j, row operand x_i
  static constexpr fused_pass PASS = fused_pass::forward;
  static constexpr int NSRC = 1, NROW = 1, RING4 = 4, RING8 = 4;
  static constexpr bool PER_ENTRY = false, ACCUMULATE = false;
  // Two entries at a time, us one / two: R-MAT, 60 k rows, 1.5 M entries: 128 columns 63.4 / 60.0, 256 127 / 111; 200 k, 4 M: 164.6 / 162.2, 390 / 388; not with
  // 16 lanes: 300 k, 3 M, 64 columns 75.1 / 76.5, 1 M, 17 M: 32 193 / 197, 64 378 / 382.
  static constexpr int NDOT = OP != ISP_OP_ONE ? 1 : 0, NSCAL = 1, PAIR_LPG = 32;
  using args = g_args1;
  template <int W, bool TAIL>
  __device__ static inline void dots(const float (&x)[1][W], const float (&r)[1][W], const lane_cols<W / 4, TAIL>& lc, float* p) {
    p[0] = dotw<W, TAIL>(r[0], x[0], lc);
  }
  __device__ static inline void scalars(const float* t, float* s) {
    float dsg;
    edge_fn(OP, t[0], s[0], dsg);
  }
  template <int W>
  __device__ static inline void apply(float a, const float* s, const float (&x)[1][W], float (&acc)[W]) {
    const float w = a * s[0];
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
