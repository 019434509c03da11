// Grouped FusedMM passes: the parts their translation units share (one unit per policy: they are compiled for every
// width class, edge function and tail, which takes a minute each).
#pragma once
#include "grouped_ops.h"

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

// Up to 16 columns four lanes hold a row, and a step serves 16 entries instead of 8, half of whose lanes were idle; below this size, where a
// launch is the time of its chains, the longer start of 16 runs counts.  us with 8 / 4 lanes, forward and backward (R-MAT, directed, 8 columns): 3 k
// rows, 30 k entries 5.3 / 5.5, 12.0 / 12.0; 10 k, 100 k: 6.3 / 6.1, 15.0 / 13.3; 20 k, 300 k: 10.1 / 9.0, 24.7 / 21.2; 100 k, 1 M: 17.9 / 14.7,
// 49.5 / 41.3; 60 k, 2.8 M: 35.2 / 28.0, 96.6 / 77.5 (16 columns 36.0 / 29.8, 99.1 / 81.0; symmetric 65.4 / 47.3); 200 k, 8 M: 91.7 / 73.5, 250 / 199; 230 k,
// 60 M: 521 / 413, 1489 / 1140; uniform, 500 k, 8 M, which waits for its gathers: 117.2 / 116.6, 385 / 386.
constexpr int64_t FUSED_NARROW_NNZ = 64 << 10;

// One or two float4 per lane.  Two halve the lanes per dot product, so a step covers twice the entries with one
// lane-reduction stage and one evaluation of the edge function less per entry, but hold twice the registers and load
// the row operand with every step.  With as few entries as the chip's wavefronts finish in a few rounds the length of their runs counts,
// and two it is: beyond 128 columns below 1 Mi entries, beyond 64 below 3/4 Mi (us, one / two, forward and backward: R-MAT, 1.2 k rows, 13 k entries, 227
// columns 17.0 / 10.9, 46.7 / 29.4; 12 k, 482 k, 144: 42.0 / 33.6, 77 / 62; 11 k, 899 k, 203: 78 / 58, 149 / 126; 3.8 k, 120 k, 96: 11.7 / 9.7, 18.2 /
// 15.5; uniform, 6 k, 196 k, 176: 22.4 / 19.3, 42.0 / 36.5; 7 k, 406 k, 72: 23.3 / 19.6, 51.6 / 36.6; but 133 k, 1.04 M, 200: 118 / 113, 233 / 254;
// 68 k, 1.07 M, 123: 54.3 / 61.4, 176 / 196; 27 k, 560 k, 60: 19.2 / 21.1, 53.6 / 55.2).  Larger ones have one everywhere (128 columns, us, one / two: forward on 2.4 M entries
// 113 / 116, on 16.9 M 823 / 858, backward 240 / 266, 2830 / 2936) except where rows average 200 entries and nearly
// all work lies in hub segments (115 M entries: 3077 / 2764, backward 7697 / 6860).  ISP_FUSED_W=4 / 8 forces
// either (d > 32).
inline bool two_vectors(const isp_csr* A, int d) {
  if (A->tune.fused_w) return A->tune.fused_w == 8;
  const int64_t nnz = A->info.nnz, live_rows = A->info.n_rows - A->info.bin_rows[0];
  if (live_rows > 0 && nnz >= 200 * live_rows) return true;
  return d > 128 ? nnz < (1 << 20) : d > 64 && nnz < (3 << 18);
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
  if (d <= 16 && A->info.nnz >= FUSED_NARROW_NNZ) return run_grouped<P, 4, 4, true>(A, pa, d, Y, ldy, s);
  if (d <= 32) return run_grouped<P, 8, 4, true>(A, pa, d, Y, ldy, s);
  if (!two_vectors(A, d)) {
    if (d <= 64) return run_grouped<P, 16, 4, true>(A, pa, d, Y, ldy, s);
    if (d <= 128) return run_grouped<P, 32, 4, true>(A, pa, d, Y, ldy, s);
    return run_grouped<P, 64, 4, true>(A, pa, d, Y, ldy, s);
  }
  if (d <= 64) return run_grouped<P, 8, 8, true>(A, pa, d, Y, ldy, s);
  if (d <= 128) return run_grouped<P, 16, 8, true>(A, pa, d, Y, ldy, s);
  return run_grouped<P, 32, 8, true>(A, pa, d, Y, ldy, s);
}

}  // namespace
