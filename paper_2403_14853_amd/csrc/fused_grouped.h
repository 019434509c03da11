// Grouped FusedMM passes: the parts their translation units share (one unit per policy: they are compiled for every
// width class, edge function and tail, which takes a minute each).
#pragma once
#include "grouped_ops.h"
#include "lane_rule.h"

namespace {
using namespace isp_dev;

// (hardware exponential and reciprocal, about 1 ulp each; exp overflow gives 1 / inf = 0)
__device__ inline float sigmoidf_fast(float z) { return __builtin_amdgcn_rcpf(1.f + __expf(-z)); }

// Edge function s = f(z) and its derivative; op is wave-uniform (ISP_OP_SIGMOID / _DOT / _ONE).
// The grouped kernels pass it as a compile-time constant, the generic ones at run time.
__device__ inline void edge_fn(int op, float z, float& s, float& ds) {
  if (op == ISP_OP_SIGMOID) { s = sigmoidf_fast(z); ds = s * (1.f - s); }
  else if (op == ISP_OP_DOT) { s = z; ds = 1.f; }
  else { s = 1.f; ds = 0.f; }
}

template <int VEC, int T, bool ACC>
__global__ void __launch_bounds__(ISP_WG) k_fused_fixup(isp_view A, int d, float* __restrict__ Y, int64_t ldy) {
  hub_fixup<VEC, T, ACC>(A, d, 0, Y, ldy);
}

// The grouped kernels' (rows of at most one partial row): the order in which a launch that finishes its hub rows adds them.
template <bool ACC>
__global__ void __launch_bounds__(ISP_WG) k_fused_fixup_wg(isp_view A, int d, float* __restrict__ Y, int64_t ldy) {
  hub_fixup_wg<4, 1, false, ACC>(A, d, 0, Y, ldy, 0);
}

template <class P, int LPG, int W, bool ADDR32, bool TAIL, bool FINISH>
__global__ void __launch_bounds__(ISP_WG) k_fused_grouped(isp_view A, const int64_t* __restrict__ indptr,
                                                          const int32_t* __restrict__ indices,
                                                          const float* __restrict__ values, typename P::args pa, int d,
                                                          float* __restrict__ Y, int64_t ldy) {
  __shared__ rn_lds lds;
  fused_grouped_item<P, LPG, W, ADDR32, TAIL, FINISH>(A, indptr, indices, values, pa, d, Y, ldy, lds);
}

// LPG lanes with W floats each span the feature width: W * LPG >= d.
// A32: every gather offset fits 32 bits.
template <class P, int LPG, int W, bool A32>
isp_status run_grouped(const isp_csr* A, const typename P::args& pa, int d, float* Y, int64_t ldy, hipStream_t s) {
  const isp_view& v = A->v;
  const bool finish = A32 && hf_pays(A, v, LPG);
  const int n_items = v.n_blocks + v.n_seg;
  if (n_items > 0) {
    const unsigned grid = (unsigned)((n_items + ISP_WAVES_PER_WG - 1) / ISP_WAVES_PER_WG);
#define ISP_GO(TL, FN) k_fused_grouped<P, LPG, W, A32, TL, FN><<<grid, ISP_WG, 0, s>>>(v, v.indptr, v.indices, v.values, pa, d, Y, ldy)
    if (d % 4) { if (finish) ISP_GO(true, A32); else ISP_GO(true, false); }
    else { if (finish) ISP_GO(false, A32); else ISP_GO(false, false); }
#undef ISP_GO
    ISP_LAUNCH_CHECK();
  }
  if (v.n_hub > 0 && !finish) {
    k_fused_fixup_wg<P::ACCUMULATE><<<(unsigned)v.n_hub, ISP_WG, 0, s>>>(v, d, Y, ldy);
    ISP_LAUNCH_CHECK();
  }
  return ISP_OK;
}

// P's shape on A (lane_rule.h); ISP_FUSED_W=4 / 8 forces one or two vectors (d > 32).
template <class P>
bool two_vectors(const isp_csr* A, int d) {
  if (A->tune.fused_w) return A->tune.fused_w == 8;
  return fused_two_vectors(P::PASS, d, A->info.n_rows, A->info.n_rows - A->info.bin_rows[0], A->info.nnz);
}
template <class P>
isp_status run_grouped_d(const isp_csr* A, const typename P::args& pa, int d, float* Y, int64_t ldy, hipStream_t s) {
  bool a32 = true;  // (the matrix is square: row operands have as many rows as gathered ones)
  for (int k = 0; k < P::NSRC; ++k) a32 = a32 && fused_offsets_fit_32(A->v.n_cols, pa.lds_[k], d);
  for (int k = 0; k < P::NROW; ++k) a32 = a32 && fused_offsets_fit_32(A->v.n_rows, pa.ldr[k], d);
  if (!a32) {  // operands of 4 GB and more: 64-bit addresses, two float4 per lane at every width
    if (d <= 64) return run_grouped<P, 8, 8, false>(A, pa, d, Y, ldy, s);
    if (d <= 128) return run_grouped<P, 16, 8, false>(A, pa, d, Y, ldy, s);
    return run_grouped<P, 32, 8, false>(A, pa, d, Y, ldy, s);
  }
  if (fused_four_lanes(P::PASS, d, A->info.nnz, A->v.n_hub)) return run_grouped<P, 4, 4, true>(A, pa, d, Y, ldy, s);
  if (d <= 32) return run_grouped<P, 8, 4, true>(A, pa, d, Y, ldy, s);
  if (!two_vectors<P>(A, d)) {
    if (d <= 64) return run_grouped<P, 16, 4, true>(A, pa, d, Y, ldy, s);
    if (d <= 128) return run_grouped<P, 32, 4, true>(A, pa, d, Y, ldy, s);
    return run_grouped<P, 64, 4, true>(A, pa, d, Y, ldy, s);
  }
  if (d <= 64) return run_grouped<P, 8, 8, true>(A, pa, d, Y, ldy, s);
  if (d <= 128) return run_grouped<P, 16, 8, true>(A, pa, d, Y, ldy, s);
  return run_grouped<P, 32, 8, true>(A, pa, d, Y, ldy, s);
}

}  // namespace
