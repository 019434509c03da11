// CSR ingest: structural validation, degree classes and the wavefront work partition.
//
// Rows are classed by degree (0 | 1..4 | 5..32 | 33..hub_t | hub).  Short rows are grouped
// into contiguous row blocks of about block_cost units, one unit per nonzero plus one per row
// (a row's output write costs about as much as one gathered input row).  Hub rows
// (degree > hub_t) never share a block; each is cut into segments of at most seg_len nonzeros whose
// partial sums are combined later in a fixed order.  On large matrices a hub row is cut first where its (sorted) columns
// cross the boundaries of column bands, so that a segment gathers dense rows from one band only (which matrices:
// partition_sizes.h), and the segments are scheduled in order of their first column: the whole chip then works on one band of the
// dense operand at a time and the L2 caches hold that band's frequently used rows instead of a sample
// of all of them.
// Everything here is integer work and runs once per graph (balanced scheduling: paper Section 1(b); CSR
// operand: Section 3.5).
#include <limits.h>
#include <new>
#include "digit_scan.h"
#include "host_slot.h"
#include "hub_rule.h"
#include "stage_rule.h"

namespace {
using namespace isp_dev;
using namespace isp_part;

struct build_counters {
  unsigned long long bin_rows[5];
  unsigned long long bin_nnz[5];
  unsigned long long max_degree;
  int err;            // bit 0: indptr malformed, bit 1: column index out of range
  int n_blocks, n_hub, n_seg;
};

constexpr size_t PARTIAL_ROW = ISP_PARTIAL_TILE * sizeof(float);
constexpr int CUT_COUNT = 16;  // wavefronts' worth of entries that cutting a hub row looks at first
constexpr int CUT_LAST = 8;    // candidates of a cut that are looked at together

// Matrices up to this size have everything about their partition enqueued in one go (see build_partition).
constexpr int64_t SMALL_NNZ = 4 << 20;

}  // namespace

isp_tuning isp_read_tuning() {
  isp_tuning t;
  t.no_grouped = getenv("ISP_NO_GROUPED") != nullptr;
  t.sddmm_one_pass = getenv("ISP_SDDMM_ONE_PASS") != nullptr;
  const int lpg = env_int("ISP_SPMM_LPG", 0, 0, 64);
  t.spmm_lpg = (lpg == 4 || lpg == 8 || lpg == 16 || lpg == 32 || lpg == 64) ? lpg : 0;
  const int tile = env_int("ISP_SPMM_TILE", 0, 0, 256);
  t.spmm_tile = (tile == 64 || tile == 128 || tile == 256) ? tile : 0;
  t.stage_min = isp_stage::read_min();
  t.wide_groups = env_int("ISP_WIDE_GROUPS", 0, 0, 4);
  t.no_mirror = getenv("ISP_NO_MIRROR") != nullptr;
  const int fw = env_int("ISP_FUSED_W", 0, 0, 8);
  t.fused_w = (fw == 4 || fw == 8) ? fw : 0;
  return t;
}

int isp_wave_slots() {
  constexpr int MAX_DEV = 64;
  static int cached[MAX_DEV] = {};  // 0 = not asked yet (racing first calls store the same number)
  constexpr int fallback = 256 * 16;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); return fallback; }
  if (dev >= 0 && dev < MAX_DEV && cached[dev]) return cached[dev];
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) {
    (void)hipGetLastError();
    return fallback;
  }
  const int slots = cus * 16;  // 4 SIMDs per compute unit x the 4 waves per SIMD the kernels are built for
  if (dev >= 0 && dev < MAX_DEV) cached[dev] = slots;
  return slots;
}

namespace {

__device__ __forceinline__ int64_t wave_uniform(int64_t v) {
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)v), hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(v >> 32));
  return (int64_t)((unsigned long long)hi << 32 | lo);
}

// Pieces of a hub row: its entries [a, b) cut where the columns cross band boundaries.  A row of degree
// deg is cut into br = the largest power of two <= min(bands, deg / min_piece) coarse bands, each made of
// bands / br fine bands of width ceil(n_cols / bands).  The whole wavefront calls this with the same row
// (a, b wave-uniform): lane j < br gets piece j as [*first, *last), the other lanes an empty piece.  Every
// lane finds one cut position by searching, which assumes ascending columns; on a row that is not sorted the positions are made monotone, so they are still valid cuts (inside the row, in order) and only
// the scheduling benefit is lost, never correctness.
__device__ inline void wave_hub_pieces(const int32_t* __restrict__ indices, int64_t a, int64_t b, int64_t n_cols,
                                       const partition_params& pp, int lane, int* samples, int64_t* first, int64_t* last) {
  // (the row is the wavefront's: kept in scalar registers; positions and columns fit 32 bits, relative to the row from here on)
  a = wave_uniform(a);
  b = wave_uniform(b);
  const int deg = (int)(b - a);
  const int32_t* __restrict__ row = indices + a;
  const int br = hub_bands(deg, pp);
  const unsigned bw = ((unsigned)n_cols + pp.bands - 1u) / (unsigned)pp.bands;
  const int step = pp.bands / br;
  // cut j = number of the row's columns below j * step * bw; cut 0 = 0, cuts >= br = deg
  const unsigned target = (unsigned)lane * step * bw;  // (below 2^31 + bands for the lanes that search)
  int lo = lane >= br ? deg : 0;
  if (br > 1) {
    // CUT_COUNT * 64 evenly spaced entries (a short row whole) in one trip to memory, searched in LDS, leave each cut a
    // range of `gap` entries; a binary search from the start would be a chain of a dozen trips, counting the samples
    // below each cut with ballots some 2,000 instructions per row (with that, 64-bit positions and 64-bit sums, the two
    // passes that cut rows took 23.6 and 15.7 us on 1 M entries, now 15 and 10).
    const int gap = (int)(((unsigned)deg + CUT_COUNT * ISP_WAVE - 1u) / (CUT_COUNT * ISP_WAVE));
    const int ns = (int)((unsigned)(deg + gap - 1) / (unsigned)gap);
    int c[CUT_COUNT];
    const unsigned lane_byte = (unsigned)lane * ((unsigned)gap * 4u);  // (a scalar base and one offset for all: gap is 2^21 at most)
#pragma unroll
    for (int k = 0; k < CUT_COUNT; ++k) {
      const char* from = reinterpret_cast<const char*>(row + (int64_t)k * ISP_WAVE * gap);
      c[k] = 0;
      if (k * ISP_WAVE + lane < ns) c[k] = *reinterpret_cast<const int32_t*>(from + lane_byte);
    }
    wave_lds_sync();  // (the row before this one has been searched)
#pragma unroll
    for (int k = 0; k < CUT_COUNT; ++k) samples[k * ISP_WAVE + lane] = c[k];
    wave_lds_sync();
    const bool mine = lane > 0 && lane < br;
    int n = 0;  // samples below the cut
    for (int st = 1 << (31 - __clz(ns)); st > 0; st >>= 1)
      if (mine && n + st <= ns && (unsigned)samples[n + st - 1] < target) n += st;
    int hi = lo;
    if (mine) {
      lo = n > 0 ? (n - 1) * gap + 1 : 0;
      hi = n < ns ? n * gap : deg;
    }
    while (__any(hi - lo > CUT_LAST)) {
      if (hi - lo > CUT_LAST) {
        const int mid = (int)(((unsigned)lo + (unsigned)hi) >> 1);
        if ((unsigned)row[mid] < target) lo = mid + 1; else hi = mid;
      }
    }
    if (__any(lo < hi)) {  // the last few candidates in one trip
      int below = 0;
#pragma unroll
      for (int k = 0; k < CUT_LAST; ++k) below += lo + k < hi && (unsigned)row[lo + k] < target;
      lo += below;
    }
  }
  int cut = lo;
#pragma unroll
  for (int o = 1; o < ISP_WAVE; o <<= 1) {  // running maximum over the lanes: monotone cuts
    const int t = __shfl_up(cut, o);
    if (lane >= o && t > cut) cut = t;
  }
  int next = __shfl_down(cut, 1);
  if (lane == ISP_WAVE - 1) next = deg;  // (the last lane has no neighbour; it holds a piece only with 64 bands)
  *first = lane < br ? a + cut : b;
  *last = lane < br ? a + next : b;
}

__device__ inline int degree_bin(long long deg, int hub_t) {
  if (deg <= 0) return 0;
  if (deg > hub_t) return 4;
  if (deg <= 4) return 1;
  if (deg <= 32) return 2;
  return 3;
}

// The partition's bookkeeping runs in three passes over the rows, each a tile of consecutive rows per workgroup: the
// first leaves every tile's sums, the later ones start by adding up the sums of the tiles before theirs (a few
// thousand numbers at most) instead of waiting for a scan in launches of its own.  A launch of this size takes about
// 5 us whatever it does, and a graph that is seen once (1 M entries) spent 632 us in 93 of them.
constexpr int64_t MAX_TILES = 4096;

// What pass 1 finds out about a tile besides the sums, STATS numbers per tile: rows per class, entries per class, longest
// row.  (Added up in pass 2: hundreds of workgroups with a dozen atomics each on one line took 25 us.)
constexpr int STATS = 11;

struct row_tiles {
  int64_t rows;    // per tile
  int n;           // tiles
  int64_t* cost;   // sums per tile
  int32_t *hub, *seg, *mark;
  unsigned long long* stats;  // [STATS][MAX_TILES]
  int32_t* err;    // build_counters::err of every workgroup of pass 1, MAX_TILES at most
};

// Rows per wavefront: the workgroup's wavefronts turn to its hub rows one after the other, a few trips to memory each, so
// small matrices spread their rows thin.
constexpr int RPW_SMALL = 16, RPW_LARGE = ISP_WAVE;

// Pass 1.  Per row: degree, class, cost, segment count; indptr checks; column indices in [0, n_cols) (check).  Workgroups beyond the
// tiles only check indices.
template <int RPW>
__global__ void __launch_bounds__(BS_THREADS, 7) k_row_pass(const int64_t* __restrict__ indptr,
                                                  const int32_t* __restrict__ indices, int64_t n_rows, int64_t n_cols,
                                                  int64_t nnz, partition_params pp, bool check, row_tiles T,
                                                  int32_t* __restrict__ cost, int32_t* __restrict__ hubflag,
                                                  int32_t* __restrict__ nseg, float* __restrict__ inv_len) {
  // The tile's numbers: STATS of them, then cost, segments, hub rows (a tile's cost: nnz + two units per row, below 2^32).  Added up
  // in LDS: sums over the lanes held 14 values per lane and with them four workgroups to a compute unit instead of seven, too few for all
  // tiles of 100 k rows at once (1 M entries: 14.5 us, now 11.2).  Sixteen copies of each: rows of one class otherwise add to
  // one address lane after lane (building 2.4 M uniform rows, 10 M entries: sums over the lanes 218 us, one copy 257, sixteen 171; 1 M rows, 4 M entries 93 / 85 / 70).
  constexpr int COST = STATS, SEGS = STATS + 1, HUBS = STATS + 2, SUM_COPIES = 16;
  __shared__ unsigned s_sum[STATS + 3][SUM_COPIES];
  __shared__ int s_hubs[BS_THREADS / ISP_WAVE];
  __shared__ int64_t s_ha[BS_THREADS], s_hb[BS_THREADS];  // the step's hub rows, [a, b), and their segments
  __shared__ int s_ns[BS_THREADS];
  __shared__ int s_samples[BS_THREADS / ISP_WAVE][CUT_COUNT * ISP_WAVE];
  __shared__ int s_err[BS_THREADS / ISP_WAVE];
  const int lane = threadIdx.x & (ISP_WAVE - 1), w = threadIdx.x / ISP_WAVE;
  const int64_t r0 = (int64_t)blockIdx.x * T.rows, r1 = r0 + T.rows < n_rows ? r0 + T.rows : n_rows;
  constexpr int STEP = (BS_THREADS / ISP_WAVE) * RPW;  // rows at a time
  const bool tile = (int)blockIdx.x < T.n;
  auto row_of = [&](int64_t base) { return base + w * RPW + lane; };
  auto in_tile = [&](int64_t i) { return tile && lane < RPW && i < r1; };
  // (the first step's offsets are on their way while the indices are looked at)
  const bool valid0 = in_tile(row_of(r0));
  const int64_t a0 = valid0 ? indptr[row_of(r0)] : 0, b0 = valid0 ? indptr[row_of(r0) + 1] : 0;
  int my_err = 0;
  if (check) {
    bool bad = false;
    const int64_t all = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < nnz; p += all * 4) {
      int32_t c[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) c[u] = p + u * all < nnz ? indices[p + u * all] : 0;
#pragma unroll
      for (int u = 0; u < 4; ++u) bad |= (c[u] < 0 || c[u] >= n_cols) && p + u * all < nnz;
    }
    my_err = bad ? 2 : 0;
  }
  auto report = [&]() {  // what this workgroup found wrong
    const int e = (__any(my_err & 1) ? 1 : 0) | (__any(my_err & 2) ? 2 : 0);
    if (lane == 0) s_err[w] = e;
    __syncthreads();
    if (threadIdx.x == 0) T.err[blockIdx.x] = s_err[0] | s_err[1] | s_err[2] | s_err[3];
  };
  if (!tile) { report(); return; }
  static_assert((STATS + 3) * SUM_COPIES <= BS_THREADS, "a copy per thread");
  const int own_sum = (int)threadIdx.x / SUM_COPIES, own_copy = (int)threadIdx.x % SUM_COPIES;
  if (own_sum < STATS + 3) s_sum[own_sum][own_copy] = 0;  // (a barrier comes before the first is added to)
  for (int64_t base = r0; base < r1; base += STEP) {  // (the workgroup stays together)
    const int64_t i = row_of(base);
    const bool valid = in_tile(i);
    int64_t a = a0, b = b0;
    if (base > r0) {
      a = valid ? indptr[i] : 0;
      b = valid ? indptr[i + 1] : 0;
    }
    long long deg = b - a;
    if (valid && (deg < 0 || a < 0 || b > nnz || (i == 0 && a != 0) || (i == n_rows - 1 && b != nnz))) { my_err |= 1; deg = 0; }
    const bool hub = deg > pp.hub_t;
    int ns = 0;
    if (pp.bands == 1) {  // (segments of one length: nothing to look for)
      __syncthreads();    // (the sums are zero)
      if (hub) ns = (int)((unsigned)(deg + pp.seg_len - 1) / (unsigned)pp.seg_len);
    } else {
      // the step's hub rows, shared out over the wavefronts
      const unsigned long long hm = __ballot(hub);
      if (lane == 0) s_hubs[w] = __popcll(hm);
      __syncthreads();
      int h0 = 0, n_hubs = 0;
#pragma unroll
      for (int ww = 0; ww < BS_THREADS / ISP_WAVE; ++ww) { h0 += ww < w ? s_hubs[ww] : 0; n_hubs += s_hubs[ww]; }
      const int hx = h0 + __popcll(hm & ((1ull << lane) - 1ull));
      if (hub) { s_ha[hx] = a; s_hb[hx] = b; }
      __syncthreads();
      for (int h = w; h < n_hubs; h += BS_THREADS / ISP_WAVE) {
        int64_t first, last;
        wave_hub_pieces(indices, s_ha[h], s_hb[h], n_cols, pp, lane, s_samples[w], &first, &last);
        int cnt = (int)((unsigned)(last - first + pp.seg_len - 1) / (unsigned)pp.seg_len);
#pragma unroll
        for (int o = 1; o < ISP_WAVE; o <<= 1) cnt += __shfl_xor(cnt, o);
        if (lane == 0) s_ns[h] = cnt;
      }
      __syncthreads();
      if (hub) ns = s_ns[hx];
    }
    if (!valid) continue;
    const int32_t c = hub ? 0 : (int32_t)deg + pp.row_cost;
    cost[i] = c;
    hubflag[i] = hub ? 1 : 0;
    nseg[i] = ns;
    inv_len[i] = deg > 0 ? 1.f / (float)deg : 0.f;
    const int bin = degree_bin(deg, pp.hub_t);
    atomicAdd(&s_sum[bin][own_copy], 1u);
    atomicAdd(&s_sum[5 + bin][own_copy], (unsigned)deg);
    atomicMax(&s_sum[10][own_copy], (unsigned)deg);
    if (hub) {
      atomicAdd(&s_sum[SEGS][own_copy], (unsigned)ns);
      atomicAdd(&s_sum[HUBS][own_copy], 1u);
    } else {
      atomicAdd(&s_sum[COST][own_copy], (unsigned)c);
    }
  }
  report();  // (a barrier)
  unsigned v = own_sum < STATS + 3 ? s_sum[own_sum][own_copy] : 0u;
#pragma unroll
  for (int o = 1; o < SUM_COPIES; o <<= 1) {
    const unsigned u = __shfl_xor(v, o);
    v = own_sum != 10 ? v + u : (u > v ? u : v);
  }
  if (own_copy != 0) return;
  if (own_sum < STATS) T.stats[own_sum * MAX_TILES + blockIdx.x] = v;
  else if (own_sum == COST) T.cost[blockIdx.x] = v;
  else if (own_sum == SEGS) T.seg[blockIdx.x] = (int)v;
  else if (own_sum == HUBS) T.hub[blockIdx.x] = (int)v;
}

// Pass 2.  Where blocks begin: block b at the first row whose cumulative short-row cost reaches b * block_cost, and at
// every hub row, at the row after one and at force_row (if inside the matrix; the derived matrix of the packed SpMM
// layout keeps blocks of whole rows and blocks of row pieces apart that way).
__global__ void __launch_bounds__(BS_THREADS) k_mark_rows(const int32_t* __restrict__ cost,
                                                          const int32_t* __restrict__ hubflag, int64_t n_rows,
                                                          int block_cost, int64_t force_row, row_tiles T, int n_err,
                                                          int32_t* __restrict__ mark, build_counters* __restrict__ ctr,
                                                          const int* __restrict__ flag, int* __restrict__ host_flag) {
  // More workgroups than tiles: what the counters tell the caller (pass 3 adds the counts), one number each (one
  // workgroup for all of them was what the launch waited for: 9.4 us on 1 M entries, now 6), and a flag that earlier launches left on the
  // device, if there is one, for the host.
  if ((int)blockIdx.x >= T.n) {
    const int k = (int)blockIdx.x - T.n - 1;
    if (k < 0) {
      int err = 0;
#pragma unroll 8
      for (int i = threadIdx.x; i < n_err; i += BS_THREADS) err |= T.err[i];
      const int err1 = __syncthreads_or(err & 1), err2 = __syncthreads_or(err & 2);
      if (threadIdx.x == 0) {
        ctr->err = (err1 ? 1 : 0) | (err2 ? 2 : 0);
        if (host_flag) *host_flag = *flag;
      }
      return;
    }
    __shared__ unsigned long long part[BS_THREADS / ISP_WAVE];
    const bool add = k < 10;  // (the longest row is the largest of them)
    unsigned long long v = 0;
#pragma unroll 8
    for (int t = threadIdx.x; t < T.n; t += BS_THREADS) {
      const unsigned long long u = T.stats[k * MAX_TILES + t];
      v = add ? v + u : (u > v ? u : v);
    }
#pragma unroll
    for (int o = 1; o < ISP_WAVE; o <<= 1) {
      const unsigned long long u = __shfl_xor(v, o);
      v = add ? v + u : (u > v ? u : v);
    }
    if ((threadIdx.x & (ISP_WAVE - 1)) == 0) part[threadIdx.x / ISP_WAVE] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int w = 1; w < BS_THREADS / ISP_WAVE; ++w) v = add ? v + part[w] : (part[w] > v ? part[w] : v);
      if (k < 5) ctr->bin_rows[k] = v; else if (k < 10) ctr->bin_nnz[k - 5] = v; else ctr->max_degree = v;
    }
    return;
  }
  const int64_t r0 = (int64_t)blockIdx.x * T.rows, r1 = r0 + T.rows < n_rows ? r0 + T.rows : n_rows;
  struct row_info { int cost, before, begins; };  // its cost, the one of the row before it, whether it begins a block whatever they are
  auto request = [&](int64_t i) {
    row_info f{0, 0, 0};
    if (i < r1) {
      f.cost = cost[i];
      f.begins = hubflag[i];
      if (i > 0) {
        f.before = cost[i - 1];
        f.begins |= hubflag[i - 1];
      }
      f.begins |= i == 0 || i == force_row;
    }
    return f;
  };
  row_info f = request(r0 + threadIdx.x);  // (on its way beside the tiles' sums)
  unsigned cum0 = (unsigned)(block_sum_of<int64_t>(T.cost, blockIdx.x) % block_cost);  // modulo block_cost
  int marks = 0;
  for (int64_t base = r0; base < r1; base += BS_THREADS) {
    const int64_t i = base + threadIdx.x;
    const bool valid = i < r1;
    if (base > r0) f = request(i);
    int tot;
    const unsigned cum = (cum0 + (unsigned)block_exclusive_scan<int>(f.cost, &tot)) % (unsigned)block_cost;
    if (valid) {
      // a multiple of block_cost lies in (cum - cost[i - 1], cum]: the remainder of cum is below the row before's cost
      const int m = f.begins || (int)cum < f.before;
      mark[i] = m;
      marks += m;
    }
    cum0 = (cum0 + (unsigned)tot) % (unsigned)block_cost;
  }
  int tot;
  block_exclusive_scan<int>(marks, &tot);
  if (threadIdx.x == 0) T.mark[blockIdx.x] = tot;
}

// Pass 3.  The tables: block starts, hub rows, their segments.
template <int RPW>
__global__ void __launch_bounds__(BS_THREADS, 7) k_compact(const int64_t* __restrict__ indptr, const int32_t* __restrict__ indices,
                                                 int64_t n_cols, partition_params pp, row_tiles T,
                                                 const int32_t* __restrict__ mark, const int32_t* __restrict__ hubflag,
                                                 const int32_t* __restrict__ nseg,
                                                 int64_t n_rows, int32_t* __restrict__ blk_row,
                                                 int32_t* __restrict__ hub_rows, int32_t* __restrict__ hub_seg_ptr,
                                                 int32_t* __restrict__ seg_hub, int32_t* __restrict__ seg_begin,
                                                 int32_t* __restrict__ seg_key, unsigned* __restrict__ hub_done,
                                                 build_counters* __restrict__ ctr, int64_t max_blocks, int64_t max_hub, int64_t max_seg) {
  // (asked for here, looked at behind the sums below; written by pass 2)
  const int err = ctr->err;
  const int lane = threadIdx.x & (ISP_WAVE - 1);
  __shared__ int64_t s_ha[BS_THREADS], s_hb[BS_THREADS];
  __shared__ int s_hs[BS_THREADS];
  __shared__ int s_samples[BS_THREADS / ISP_WAVE][CUT_COUNT * ISP_WAVE];
  const int64_t r0 = (int64_t)blockIdx.x * T.rows, r1 = r0 + T.rows < n_rows ? r0 + T.rows : n_rows;
  struct row_info { int mark, hub, nseg; int64_t a, b; };
  auto request = [&](int64_t base) {
    const int64_t i = base + (threadIdx.x / ISP_WAVE) * RPW + lane;
    row_info f{0, 0, 0, 0, 0};
    if (lane < RPW && i < r1) f = {mark[i], hubflag[i], nseg[i], indptr[i], indptr[i + 1]};
    return f;
  };
  row_info f = request(r0);  // (on its way beside the tiles' sums)
  int mpos0, hpos0, seg0;
  {
    unsigned long long mh = 0;  // marks and hub rows of the earlier tiles, 32 bits each
    int sg = 0;
#pragma unroll 4
    for (int t = threadIdx.x; t < (int)blockIdx.x; t += BS_THREADS) {
      mh += (unsigned long long)(unsigned)T.mark[t] << 32 | (unsigned)T.hub[t];
      sg += T.seg[t];
    }
    unsigned long long tot;
    block_exclusive_scan<unsigned long long>(mh, &tot);
    mpos0 = (int)(tot >> 32);
    hpos0 = (int)(unsigned)tot;
    block_exclusive_scan<int>(sg, &seg0);
  }
  // Rows of a malformed indptr may overlap: their segments together can wrap the 32-bit sums, whatever the tables' bounds.
  if (err & 1) return;  // (the host reports ISP_EBADCSR)
  for (int64_t base = r0; base < r1; base += (BS_THREADS / ISP_WAVE) * RPW) {
    const int64_t i = base + (threadIdx.x / ISP_WAVE) * RPW + lane;
    if (base > r0) f = request(base);  // (no early exit: the wavefront handles its hub rows together)
    const int m = f.mark;
    const bool hub = f.hub;
    // one scan for the three positions (at most 256 marks and hub rows here)
    unsigned long long tot;
    const unsigned long long pos = block_exclusive_scan<unsigned long long>(
        (unsigned long long)m << 48 | (unsigned long long)(hub ? 1 : 0) << 32 | (unsigned)(hub ? f.nseg : 0), &tot);
    const int mpos = mpos0 + (int)(pos >> 48), h = hpos0 + (int)(pos >> 32 & 0xffff), s0 = seg0 + (int)(unsigned)pos;
    mpos0 += (int)(tot >> 48);
    hpos0 += (int)(tot >> 32 & 0xffff);
    seg0 += (int)(unsigned)tot;
    if (m && mpos < max_blocks) blk_row[mpos] = (int32_t)i;
    const int64_t a = hub ? f.a : 0, b = hub ? f.b : 0;
    if (hub && h < max_hub) {
      hub_rows[h] = (int32_t)i;
      hub_seg_ptr[h] = s0;
      for (int k = 0; k < HF_SLICES; ++k) hub_done[(int64_t)h * HF_STRIDE + k] = 0;
    }
    const int hx = (int)(pos >> 32 & 0xffff);  // the step's hub rows, shared out over the wavefronts
    if (hub) { s_ha[hx] = a; s_hb[hx] = b; s_hs[hx] = s0; }
    __syncthreads();
    const int n_hubs = (int)(tot >> 32 & 0xffff), hh0 = hpos0 - n_hubs;
    for (int hq = threadIdx.x / ISP_WAVE; hq < n_hubs; hq += BS_THREADS / ISP_WAVE) {
      const int hh = hh0 + hq, hs0 = s_hs[hq];
      auto put = [&](int64_t s, int64_t q) {  // segment s begins at entry q
        if (s >= max_seg) return;
        seg_hub[s] = hh;
        seg_begin[s] = (int32_t)q;
        seg_key[s] = indices[q];
      };
      int64_t first, last;
      if (pp.bands == 1) {  // one piece: its segments side by side (by one lane, 100 k rows, 1 M entries, one graph seen once 240 us, 217 this way)
        first = s_ha[hq];
        last = s_hb[hq];
        for (int64_t s = lane, q = first + (int64_t)lane * pp.seg_len; q < last; s += ISP_WAVE, q += (int64_t)ISP_WAVE * pp.seg_len) put(hs0 + s, q);
        continue;
      }
      wave_hub_pieces(indices, s_ha[hq], s_hb[hq], n_cols, pp, lane, s_samples[threadIdx.x / ISP_WAVE], &first, &last);
      // the row's segments, in order of position: piece by piece (lane by lane), each piece in runs of seg_len
      const int cnt = (int)((unsigned)(last - first + pp.seg_len - 1) / (unsigned)pp.seg_len);
      int inc = cnt;
#pragma unroll
      for (int o = 1; o < ISP_WAVE; o <<= 1) {
        const int t = __shfl_up(inc, o);
        if (lane >= o) inc += t;
      }
      int64_t s = (int64_t)hs0 + inc - cnt;
      for (int64_t q = first; q < last; q += pp.seg_len, ++s) put(s, q);
    }
  }
  if ((int)blockIdx.x == T.n - 1 && threadIdx.x == 0) {  // the last tile's ends are the totals
    if (mpos0 <= max_blocks) blk_row[mpos0] = (int32_t)n_rows;
    if (hpos0 <= max_hub) hub_seg_ptr[hpos0] = seg0;
    ctr->n_blocks = mpos0;
    ctr->n_hub = hpos0;
    ctr->n_seg = seg0;
  }
}

// What a work item covers, written once per handle (see isp_view::item_desc).
struct item_tables {
  const int64_t* indptr;
  const int32_t *blk_row, *hub_rows, *hub_seg_ptr, *seg_hub, *seg_begin;
  int hub_t;
};
__device__ __forceinline__ int4 block_item(const item_tables& I, int b) {
  const int row = I.blk_row[b], row_last = I.blk_row[b + 1];
  const int64_t p = I.indptr[row], p_end = I.indptr[row_last];
  const bool skip = (row_last == row + 1) && (p_end - p > I.hub_t);
  return make_int4((int)p, (int)p_end, row, skip ? -1 : row_last);
}
__device__ __forceinline__ int4 segment_item(const item_tables& I, int s) {
  const int h = I.seg_hub[s];
  const int hr = I.hub_rows[h];
  const int64_t p_end = (s + 1 < I.hub_seg_ptr[h + 1]) ? (int64_t)I.seg_begin[s + 1] : I.indptr[hr + 1];
  return make_int4(I.seg_begin[s], (int)p_end, s, hr);
}

// Up to SO_RANK segments: schedule order in one launch, every segment counting those before it (by first column, then
// number).  SO_SMALL^2 comparisons are 1.5 us of the chip's vector ALUs if all of it works on them, hence few segments per
// workgroup (5,000 segments: 11.4 us at 64, which left most of the chip idle, 7.4 at 16); a bitonic sort in one workgroup took 88 us.
// The radix sort below is three launches per digit, which beyond SO_SMALL keys cost the host more than the ranking the
// chip, up to twice as many.  us for a graph seen once (two partitions, two SpMMs), ranked / sorted / sorted in five launches per
// digit: 4 M entries, 100 k rows (some 8,200 segments) 390 / 425 / 448; 8 M, 400 k (11,242) 807 / 874 / 915; 3 M, 20 k (16,013) 353 /
// 373 / 403; 7 M, 60 k (20,754) 574 / 555; 15 M, 50 k (67,333), 32 columns - / 913 / 953.
constexpr int SO_SMALL = 8192;  // keys in LDS at a time, and the most that is ranked before their number is known on the host
constexpr int SO_RANK = 2 * SO_SMALL;
constexpr int SO_SEGS = 16;     // segments per workgroup, one per lane of 16
constexpr int SO_THREADS = 1024;
// The same launch writes the work items: a segment's place is known with its rank, and workgroups beyond the first seg_wgs,
// those of the segments, write the row blocks' (max_items bounds what the tables hold).  The counters are left in host_ctr.
// MANY: more keys than LDS takes.
template <bool MANY>
__global__ void __launch_bounds__(SO_THREADS) k_seg_rank(const int32_t* __restrict__ key,
                                                         const build_counters* __restrict__ ctr, int32_t* __restrict__ order,
                                                         item_tables I, int64_t max_items, build_counters* __restrict__ host_ctr,
                                                         int4* __restrict__ desc, int seg_wgs) {
  constexpr int PER = SO_SMALL / SO_THREADS, WAVES = SO_THREADS / ISP_WAVE, SHARES = SO_THREADS / SO_SEGS;
  __shared__ __align__(16) int keys[SO_SMALL];
  __shared__ int part[WAVES][SO_SEGS];
  if (host_ctr && blockIdx.x == 0 && threadIdx.x == 0) *host_ctr = *ctr;
  const int n = ctr->n_seg, n_blocks = ctr->n_blocks;
  // (a malformed matrix has no bounds to rely on; the rest the host sees to)
  if (ctr->err || n > seg_wgs * SO_SEGS || (int64_t)n_blocks + n > max_items) return;
  if ((int)blockIdx.x >= seg_wgs) {
    const int b = ((int)blockIdx.x - seg_wgs) * SO_THREADS + (int)threadIdx.x;
    if (b < n_blocks) desc[b] = block_item(I, b);
    return;
  }
  if ((int)blockIdx.x * SO_SEGS >= n) return;
  const int lane = threadIdx.x & (ISP_WAVE - 1), w = threadIdx.x / ISP_WAVE;
  const int s = blockIdx.x * SO_SEGS + (threadIdx.x & (SO_SEGS - 1));
  const int k = s < n ? key[s] : 0;
  int kk[PER];  // (all of them on their way together)
  auto request = [&](int base) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int j = base + u * SO_THREADS + threadIdx.x;
      kk[u] = j < n ? key[j] : INT_MAX;
    }
  };
  request(0);
  // Share h of a segment's comparisons: every SHARES-th four keys.  Keys of lower-numbered segments count when equal,
  // others only when smaller (columns are below 2^31 - 1); the four around the segment itself are put right at the end.
  const int4* __restrict__ k4 = reinterpret_cast<const int4*>(keys);
  int rank = 0;
  for (int base = 0; base < (MANY ? n : 1); base += SO_SMALL) {
    if (MANY && base > 0) __syncthreads();  // (the keys before these have been compared)
#pragma unroll
    for (int u = 0; u < PER; ++u) keys[u * SO_THREADS + threadIdx.x] = kk[u];
    __syncthreads();
    if (MANY && base + SO_SMALL < n) request(base + SO_SMALL);
    const int left = n - base < SO_SMALL ? n - base : SO_SMALL, n4 = (left + 3) / 4, own = s / 4 - base / 4;
#pragma unroll 4
    for (int j = threadIdx.x / SO_SEGS; j < n4; j += SHARES) {
      const int4 kj = k4[j];
      const int t = k + (j < own ? 1 : 0);
      rank += (kj.x < t) + (kj.y < t) + (kj.z < t) + (kj.w < t);
    }
    if (threadIdx.x < SO_SEGS && own >= 0 && own < n4)
      for (int j = own * 4; j < s - base; ++j) rank += keys[j] == k;
  }
#pragma unroll
  for (int o = SO_SEGS; o < ISP_WAVE; o <<= 1) rank += __shfl_xor(rank, o);
  if (lane < SO_SEGS) part[w][lane] = rank;
  __syncthreads();
  if (threadIdx.x < SO_SEGS && s < n) {
    rank = 0;
#pragma unroll
    for (int ww = 0; ww < WAVES; ++ww) rank += part[ww][threadIdx.x];
    order[rank] = s;
    desc[n_blocks + rank] = segment_item(I, s);
  }
}

// ---- schedule order of the segments: stable radix sort (8-bit digits) by first column -----------------
constexpr int SO_TILE = 256;
constexpr int SO_RADIX = 256;
static_assert(SO_TILE == BS_THREADS && SO_RADIX == BS_THREADS, "a digit per thread");

__global__ void __launch_bounds__(SO_TILE) k_seg_hist(const int32_t* __restrict__ key, int n_seg, int shift, int n_tiles,
                                                      int32_t* __restrict__ table) {
  __shared__ int hist[SO_RADIX];
  hist[threadIdx.x] = 0;
  __syncthreads();
  const int s = blockIdx.x * SO_TILE + threadIdx.x;
  if (s < n_seg) atomicAdd(&hist[(key[s] >> shift) & (SO_RADIX - 1)], 1);
  __syncthreads();
  table[threadIdx.x * n_tiles + blockIdx.x] = hist[threadIdx.x];
}

// val_in == NULL: the payload is the element's index (first pass)
__global__ void __launch_bounds__(SO_TILE) k_seg_scatter(const int32_t* __restrict__ key_in,
                                                         const int32_t* __restrict__ val_in, int n_seg, int shift,
                                                         int n_tiles, const int32_t* __restrict__ table_scanned,
                                                         const int32_t* __restrict__ digit_total,
                                                         int32_t* __restrict__ key_out, int32_t* __restrict__ val_out) {
  __shared__ int digits[SO_TILE], start[SO_RADIX];  // start: elements with a smaller digit
  int all;
  start[threadIdx.x] = block_exclusive_scan<int>(digit_total[threadIdx.x], &all);
  const int s = blockIdx.x * SO_TILE + threadIdx.x;
  const int key = s < n_seg ? key_in[s] : 0;
  const int dg = s < n_seg ? (key >> shift) & (SO_RADIX - 1) : -1;
  digits[threadIdx.x] = dg;
  __syncthreads();
  if (dg < 0) return;
  int rank = 0;  // earlier elements of this tile with the same digit
  for (int t = 0; t < (int)threadIdx.x; ++t) rank += (digits[t] == dg);
  const int dst = start[dg] + table_scanned[dg * n_tiles + blockIdx.x] + rank;
  key_out[dst] = key;
  val_out[dst] = val_in ? val_in[s] : s;
}

// All work items at once, for partitions whose counts the host knows.
__global__ void __launch_bounds__(256) k_item_desc(item_tables I, int n_blocks, const int32_t* __restrict__ seg_order, int n_seg,
                                                   int4* __restrict__ desc) {
  const int item = blockIdx.x * blockDim.x + threadIdx.x;
  if (item < n_blocks) desc[item] = block_item(I, item);
  else if (item < n_blocks + n_seg) desc[item] = segment_item(I, seg_order[item - n_blocks]);
}

// ---- the derived matrix of the packed SpMM layout ------------------------------------------------------
// Rows longer than mid_t ("cut rows") are cut into column-band pieces exactly like hub rows, but with a lower
// threshold and smaller pieces, and the pieces - far too short to be work items of their own - become the rows
// of a derived CSR that is appended, in schedule order (by first column), to a copy of the short rows:
//   rows [0, n)        : the matrix's own rows, the cut ones left empty
//   rows [n, n + n_pc) : the pieces, piece k being segment seg_order[k] of the cut partition
// The derived matrix has short rows only, so the ordinary row blocks pack several pieces into every
// full-sized work item; a piece's sum goes to the partial row of its segment and the fixed-order fix-up adds a
// cut row's pieces as it does a hub row's segments.

// lengths of the short part's rows (0 for a cut row)
__global__ void __launch_bounds__(256) k_short_len(const int64_t* __restrict__ indptr, const int32_t* __restrict__ hubflag,
                                                   int64_t n_rows, int32_t* __restrict__ len) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_rows) len[i] = hubflag[i] ? 0 : (int32_t)(indptr[i + 1] - indptr[i]);
}

// lengths of the pieces in schedule order
__global__ void __launch_bounds__(256) k_piece_len(const int64_t* __restrict__ indptr, const int32_t* __restrict__ hub_rows,
                                                   const int32_t* __restrict__ hub_seg_ptr,
                                                   const int32_t* __restrict__ seg_hub,
                                                   const int32_t* __restrict__ seg_begin,
                                                   const int32_t* __restrict__ seg_order, int n_seg,
                                                   int32_t* __restrict__ len) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n_seg) return;
  const int s = seg_order[k];
  const int h = seg_hub[s];
  const int64_t end = (s + 1 < hub_seg_ptr[h + 1]) ? (int64_t)seg_begin[s + 1] : indptr[hub_rows[h] + 1];
  len[k] = (int32_t)(end - seg_begin[s]);
}

// row offsets of the derived matrix: the short part's scan, then the pieces' scan behind it
__global__ void __launch_bounds__(256) k_join_offsets(const int64_t* __restrict__ short_scan, int64_t n_rows,
                                                      const int64_t* __restrict__ piece_scan, int64_t n_seg,
                                                      int64_t* __restrict__ indptr2) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_rows) indptr2[i] = short_scan[i];
  else if (i <= n_rows + n_seg) indptr2[i] = short_scan[n_rows] + piece_scan[i - n_rows];
}

// Copy of the short rows' entries.  One thread per stored entry of the source matrix; the workgroup's tile of
// consecutive entries spans a narrow range of rows, found once per tile, in which each thread then searches.
constexpr int CP_TILE = 1024;
__global__ void __launch_bounds__(256) k_copy_short(const int64_t* __restrict__ indptr, const int32_t* __restrict__ indices,
                                                    const float* __restrict__ values,
                                                    const int32_t* __restrict__ hubflag, int64_t n_rows, int64_t nnz,
                                                    const int64_t* __restrict__ indptr2, int32_t* __restrict__ indices2,
                                                    float* __restrict__ values2, int32_t* __restrict__ src_pos) {
  __shared__ int64_t s_lo, s_hi;
  const int64_t p0 = (int64_t)blockIdx.x * CP_TILE;
  if (threadIdx.x < 2) {  // last row starting at or before the tile's first / last entry
    const int64_t target = threadIdx.x == 0 ? p0 : (p0 + CP_TILE - 1 < nnz ? p0 + CP_TILE - 1 : nnz - 1);
    int64_t lo = 0, hi = n_rows;  // invariant: indptr[lo] <= target < indptr[hi]
    while (hi - lo > 1) {
      const int64_t mid = (lo + hi) >> 1;
      if (indptr[mid] <= target) lo = mid; else hi = mid;
    }
    if (threadIdx.x == 0) s_lo = lo; else s_hi = lo;
  }
  __syncthreads();
  for (int64_t p = p0 + threadIdx.x; p < p0 + CP_TILE && p < nnz; p += blockDim.x) {
    int64_t lo = s_lo, hi = s_hi + 1;  // the entry's row: last one with indptr[row] <= p
    while (hi - lo > 1) {
      const int64_t mid = (lo + hi) >> 1;
      if (indptr[mid] <= p) lo = mid; else hi = mid;
    }
    if (hubflag[lo]) continue;  // a cut row: its entries are copied piece by piece
    const int64_t q = indptr2[lo] + (p - indptr[lo]);
    indices2[q] = indices[p];
    if (values2) values2[q] = values[p];
    src_pos[q] = (int32_t)p;
  }
}

// Copy of the pieces' entries: one wavefront per piece, both sides contiguous.
__global__ void __launch_bounds__(256) k_copy_pieces(const int32_t* __restrict__ indices, const float* __restrict__ values,
                                                     const int32_t* __restrict__ seg_begin,
                                                     const int32_t* __restrict__ seg_order, int n_seg, int64_t n_rows,
                                                     const int64_t* __restrict__ indptr2, int32_t* __restrict__ indices2,
                                                     float* __restrict__ values2, int32_t* __restrict__ src_pos) {
  const int lane = threadIdx.x & (ISP_WAVE - 1);
  const int k = blockIdx.x * (blockDim.x / ISP_WAVE) + (threadIdx.x >> 6);
  if (k >= n_seg) return;
  const int64_t src = seg_begin[seg_order[k]];
  const int64_t q0 = indptr2[n_rows + k], q1 = indptr2[n_rows + k + 1];
  for (int64_t q = q0 + lane; q < q1; q += ISP_WAVE) {
    const int64_t p = src + (q - q0);
    indices2[q] = indices[p];
    if (values2) values2[q] = values[p];
    src_pos[q] = (int32_t)p;
  }
}

// out[q] = values[pos[q]].  Eight loads in flight per thread pay where one per thread fills the chip many times over
// (115 M entries in packed order: 397 us with one, 273 with eight; 40 M in the transpose's order 721 and 691; 17 M: 290 and 294; 2.4 M: 18.9 and 21.8).
constexpr int64_t GV_MANY_NNZ = 32 << 20;
template <int GV_PER_THREAD>
__global__ void __launch_bounds__(256) k_gather_values(const int32_t* __restrict__ pos, const float* __restrict__ values,
                                                       int64_t nnz, float* __restrict__ out) {
  int32_t p[GV_PER_THREAD];
  float v[GV_PER_THREAD];
  const int64_t q0 = (int64_t)blockIdx.x * (256 * GV_PER_THREAD) + threadIdx.x;
#pragma unroll
  for (int u = 0; u < GV_PER_THREAD; ++u) p[u] = q0 + u * 256 < nnz ? pos[q0 + u * 256] : 0;
#pragma unroll
  for (int u = 0; u < GV_PER_THREAD; ++u) v[u] = values[p[u]];
#pragma unroll
  for (int u = 0; u < GV_PER_THREAD; ++u)
    if (q0 + u * 256 < nnz) out[q0 + u * 256] = v[u];
}

// The same for two arrays of values with one set of positions (a symmetric pattern's packed layout serves the matrix and its
// transpose: 115 M entries, 2 x 282 us one after the other, 433 together, which reads the positions once).
constexpr int GV2_PER_THREAD = 4;
__global__ void __launch_bounds__(256) k_gather_values_pair(const int32_t* __restrict__ pos, const float* __restrict__ a,
                                                            const float* __restrict__ b, int64_t nnz,
                                                            float* __restrict__ out_a, float* __restrict__ out_b) {
  int32_t p[GV2_PER_THREAD];
  float va[GV2_PER_THREAD], vb[GV2_PER_THREAD];
  const int64_t q0 = (int64_t)blockIdx.x * (256 * GV2_PER_THREAD) + threadIdx.x;
#pragma unroll
  for (int u = 0; u < GV2_PER_THREAD; ++u) p[u] = q0 + u * 256 < nnz ? pos[q0 + u * 256] : 0;
#pragma unroll
  for (int u = 0; u < GV2_PER_THREAD; ++u) { va[u] = a[p[u]]; vb[u] = b[p[u]]; }
#pragma unroll
  for (int u = 0; u < GV2_PER_THREAD; ++u)
    if (q0 + u * 256 < nnz) { out_a[q0 + u * 256] = va[u]; out_b[q0 + u * 256] = vb[u]; }
}

static_assert(sizeof(build_counters) <= host_slot::SIZE, "the counters fit a slot");

// ---- workspace layout ------------------------------------------------------------------------------------
struct ws_layout {
  size_t counters, cost, hubflag, nseg, mark, tile_cost, tile_hub, tile_seg, tile_mark, tile_stat, tile_err;
  size_t blk_row, hub_rows, hub_seg_ptr, hub_done, seg_hub, seg_begin, seg_key[2], seg_order[2], so_table, so_total;
  size_t inv_len, item_desc, partials, total;
  int64_t max_blocks, max_hub, max_seg;
};

// The tables of one partition of a matrix with n_rows rows and nnz entries, laid out from offset `start`.
ws_layout make_layout(int64_t n_rows, int64_t nnz, const partition_params& pp, size_t start = 0,
                      bool with_partials = true) {
  ws_layout L;
  size_t off = start;
  auto take = [&](size_t bytes) { size_t o = off; off += isp_align(bytes); return o; };
  const int64_t n_bal = (nnz + (int64_t)pp.row_cost * n_rows) / pp.block_cost + 2;
  const int64_t max_hub = max_hub_rows(n_rows, nnz, pp);
  int64_t max_blocks = n_bal + 2 * max_hub + 3;
  if (max_blocks > n_rows + 1) max_blocks = n_rows + 1;
  const int64_t max_seg = max_segments(n_rows, nnz, pp);
  L.max_blocks = max_blocks; L.max_hub = max_hub; L.max_seg = max_seg;
  L.counters = take(sizeof(build_counters));
  L.cost = take((size_t)(n_rows + 1) * 4);
  L.hubflag = take((size_t)(n_rows + 1) * 4);
  L.nseg = take((size_t)(n_rows + 1) * 4);
  L.mark = take((size_t)(n_rows + 1) * 4);
  L.tile_cost = take((size_t)MAX_TILES * 8);
  L.tile_hub = take((size_t)MAX_TILES * 4);
  L.tile_seg = take((size_t)MAX_TILES * 4);
  L.tile_mark = take((size_t)MAX_TILES * 4);
  L.tile_stat = take((size_t)MAX_TILES * STATS * 8);
  L.tile_err = take((size_t)MAX_TILES * 4);
  L.blk_row = take((size_t)(max_blocks + 1) * 4);
  L.hub_rows = take((size_t)(max_hub + 1) * 4);
  L.hub_seg_ptr = take((size_t)(max_hub + 2) * 4);
  L.hub_done = take((size_t)(max_hub + 1) * HF_STRIDE * 4);
  L.seg_hub = take((size_t)(max_seg + 1) * 4);
  L.seg_begin = take((size_t)(max_seg + 1) * 4);
  for (int k = 0; k < 2; ++k) {
    L.seg_key[k] = take((size_t)(max_seg + 1) * 4);
    L.seg_order[k] = take((size_t)(max_seg + 1) * 4);
  }
  const int64_t so_tbl = (int64_t)SO_RADIX * ((max_seg + SO_TILE - 1) / SO_TILE + 1);
  L.so_table = take((size_t)(so_tbl + 1) * 4);
  L.so_total = take((size_t)SO_RADIX * 4);
  L.inv_len = take((size_t)(n_rows + 1) * 4);
  L.item_desc = take((size_t)(max_blocks + max_seg + 2) * 16);
  // (a derived matrix has no hub rows of its own, hence no partial rows)
  L.partials = take(with_partials ? (size_t)(max_seg + 1) * ISP_PARTIAL_TILE * sizeof(float) : 256);
  L.total = off;
  return L;
}

// The packed SpMM layout's share of the workspace, behind the matrix's ordinary partition.
struct packed_layout {
  ws_layout cut;      // the cut partition of the matrix itself (its partial rows are the pieces' partial rows)
  size_t indptr2, indices2, values2, src_pos, len_tmp, scan64, scan_tmp;
  size_t part2_start; // the derived matrix's partition starts here (laid out once its row count is known)
  size_t total;
};

packed_layout make_packed_layout(int64_t n_rows, int64_t nnz, bool has_values, const partition_params& p1, int mid_t,
                                 size_t start) {
  packed_layout P;
  const partition_params pc = cut_params(p1, mid_t);
  P.cut = make_layout(n_rows, nnz, pc, start);
  size_t off = P.cut.total;
  auto take = [&](size_t bytes) { size_t o = off; off += isp_align(bytes); return o; };
  const int64_t n2 = n_rows + P.cut.max_seg;
  P.indptr2 = take((size_t)(n2 + 2) * 8);
  P.indices2 = take((size_t)(nnz + 1) * 4);
  P.values2 = has_values ? take((size_t)(nnz + 1) * 4) : 0;
  P.src_pos = take((size_t)(nnz + 1) * 4);
  const int64_t longest = n_rows > P.cut.max_seg ? n_rows : P.cut.max_seg;
  P.len_tmp = take((size_t)(longest + 2) * 4);
  P.scan64 = take((size_t)(n_rows + P.cut.max_seg + 4) * 8);  // the two scans, one behind the other
  P.scan_tmp = take(isp_scan_tmp_bytes(longest + 1));
  P.part2_start = off;
  // upper bound of the derived matrix's partition
  P.total = make_layout(n2, nnz, derived_params(p1, pc), off, false).total;
  return P;
}

// Rows above this length are cut for the packed SpMM layout; 0 = no packed layout.  Chosen for large
// matrices whose dense operand is far larger than an L2 (64 Ki columns or more): there the pieces of
// mid-sized rows (too short to be work items, hence packed) gather from one band at a time like the hub
// segments do.  Measured on 233 k columns / 115 M entries: 2.50 against 2.60 ms per SpMM; on 169 k columns /
// 2.4 M entries it loses (0.125 against 0.113 ms: too few items per band), hence the lower size limit.
// ISP_MID_THRESHOLD overrides (0 disables).
// The layout costs workspace - a second copy of the entries, their source positions and one partial row per
// piece: up to about 36 bytes per stored entry - so beyond 256 Mi entries it is left out as well.
int mid_threshold(int64_t n_rows, int64_t n_cols, int64_t nnz, const partition_params& p1) {
  const int dflt = (nnz >= ((int64_t)8 << 20) && nnz <= ((int64_t)256 << 20) && n_cols >= (1 << 16)) ? 256 : 0;
  int t = env_int("ISP_MID_THRESHOLD", dflt, 0, 512);
  if (t > 0 && t < 8) t = 8;
  // the derived matrix's rows (short rows, pieces) must fit the grouped kernels' tables next to a block
  if (t > 0) {
    const partition_params c = cut_params(p1, t), dd = derived_params(p1, c);
    if (c.seg_len < 8 || dd.block_cost + dd.hub_t > 768 || dd.block_cost / dd.row_cost > 256) t = 0;
  }
  // ... and its rows (the matrix's rows plus one per piece) must stay countable in 32 bits
  if (t > 0 && n_rows + make_layout(n_rows, nnz, cut_params(p1, t)).max_seg >= 2147483646) t = 0;
  return t;
}

// One partition of a CSR matrix: every table the kernels read, in the workspace region laid out by L.
struct partition_out {
  int32_t *blk_row, *hub_rows, *hub_seg_ptr, *seg_hub, *seg_begin, *hubflag;
  const int32_t* seg_order;
  int4* item_desc;
  unsigned* hub_done;
  float* partials;
  float* inv_len;
  build_counters h;
};

isp_status build_partition(int64_t n_rows, int64_t n_cols, int64_t nnz, const int64_t* indptr, const int32_t* indices,
                           const partition_params& pp, char* base, const ws_layout& L, bool validate,
                           int64_t force_row, hipStream_t s, partition_out* out, const int* flag = nullptr,
                           int* host_flag = nullptr) {
  build_counters* ctr = (build_counters*)(base + L.counters);
  int32_t* cost = (int32_t*)(base + L.cost);
  int32_t* hubflag = (int32_t*)(base + L.hubflag);
  int32_t* nseg = (int32_t*)(base + L.nseg);
  int32_t* mark = (int32_t*)(base + L.mark);
  int32_t* blk_row = (int32_t*)(base + L.blk_row);
  int32_t* hub_rows = (int32_t*)(base + L.hub_rows);
  int32_t* hub_seg_ptr = (int32_t*)(base + L.hub_seg_ptr);
  int32_t* seg_hub = (int32_t*)(base + L.seg_hub);
  int32_t* seg_begin = (int32_t*)(base + L.seg_begin);
  int32_t* seg_key[2] = {(int32_t*)(base + L.seg_key[0]), (int32_t*)(base + L.seg_key[1])};
  int32_t* seg_ord[2] = {(int32_t*)(base + L.seg_order[0]), (int32_t*)(base + L.seg_order[1])};
  const int32_t* seg_order = seg_ord[0];
  int4* item_desc = (int4*)(base + L.item_desc);

  // Few rows: one step of thin wavefronts per workgroup; else the rows the chip has tiles for.
  const bool spread = n_rows <= MAX_TILES * (BS_THREADS / ISP_WAVE) * RPW_SMALL;
  row_tiles T;
  T.rows = spread ? (BS_THREADS / ISP_WAVE) * RPW_SMALL
                  : ((n_rows + MAX_TILES - 1) / MAX_TILES + BS_THREADS - 1) / BS_THREADS * BS_THREADS;
  T.n = n_rows > 0 ? (int)((n_rows + T.rows - 1) / T.rows) : 1;
  T.cost = (int64_t*)(base + L.tile_cost);
  T.hub = (int32_t*)(base + L.tile_hub);
  T.seg = (int32_t*)(base + L.tile_seg);
  T.mark = (int32_t*)(base + L.tile_mark);
  T.stats = (unsigned long long*)(base + L.tile_stat);
  T.err = (int32_t*)(base + L.tile_err);
  int grid1 = T.n;
  if (validate && nnz > 0) {
    const int64_t want = (nnz + 4095) / 4096;
    if (want > grid1) grid1 = want < 2048 ? (int)want : (grid1 > 2048 ? grid1 : 2048);
  }
#define ISP_GO(R)                                                                                                      \
  k_row_pass<R><<<grid1, BS_THREADS, 0, s>>>(indptr, indices, n_rows, n_cols, nnz, pp, validate, T, cost, hubflag, nseg, \
                                             (float*)(base + L.inv_len))
  if (spread) ISP_GO(RPW_SMALL); else ISP_GO(RPW_LARGE);
#undef ISP_GO
  ISP_LAUNCH_CHECK();
  k_mark_rows<<<T.n + 1 + STATS, BS_THREADS, 0, s>>>(cost, hubflag, n_rows, pp.block_cost, force_row, T, grid1, mark, ctr, flag, host_flag);
  ISP_LAUNCH_CHECK();
#define ISP_GO(R)                                                                                                     \
  k_compact<R><<<T.n, BS_THREADS, 0, s>>>(indptr, indices, n_cols, pp, T, mark, hubflag, nseg, n_rows, blk_row, hub_rows, \
                                          hub_seg_ptr, seg_hub, seg_begin, seg_key[0],              \
                                          (unsigned*)(base + L.hub_done), ctr, L.max_blocks, L.max_hub, L.max_seg)
  if (spread) ISP_GO(RPW_SMALL); else ISP_GO(RPW_LARGE);
#undef ISP_GO
  ISP_LAUNCH_CHECK();

  // Matrices of up to SMALL_NNZ entries: the rest is enqueued right behind, before the counts are known on the host (a
  // round trip through the host costs as much as three launches); more segments than the ranking takes, or a
  // partition beyond its bounds, leave it to the steps below.
  build_counters& h = out->h;
  const bool small = nnz <= SMALL_NNZ;
  const int64_t max_items = L.max_blocks + L.max_seg;
  const item_tables items{indptr, blk_row, hub_rows, hub_seg_ptr, seg_hub, seg_begin, pp.hub_t};
  host_slot slot;  // pinned: the device writes the counters there itself
  build_counters* host_ctr = small ? (build_counters*)slot.get() : nullptr;
  if (small) {
    const unsigned wgs = SO_SMALL / SO_SEGS + (unsigned)((L.max_blocks + SO_THREADS - 1) / SO_THREADS);
    k_seg_rank<false><<<wgs, SO_THREADS, 0, s>>>(seg_key[0], ctr, seg_ord[0], items, max_items, host_ctr, item_desc, SO_SMALL / SO_SEGS);
    ISP_LAUNCH_CHECK();
  }
  if (!host_ctr) ISP_HIP(hipMemcpyAsync(&h, ctr, sizeof(h), hipMemcpyDeviceToHost, s));
  ISP_HIP(hipStreamSynchronize(s));
  if (host_ctr) h = *host_ctr;
  if (h.err & 1) return isp_fail(ISP_EBADCSR, "indptr is not a monotone offset array from 0 to nnz");
  if (h.err & 2) return isp_fail(ISP_EBADCSR, "a column index lies outside [0, n_cols)");
  if (h.n_blocks > L.max_blocks || h.n_hub > L.max_hub || h.n_seg > L.max_seg)
    return isp_fail(ISP_EINVAL, "internal: partition exceeds its bounds (%d/%lld blocks, %d/%lld hubs, %d/%lld segs)",
                    h.n_blocks, (long long)L.max_blocks, h.n_hub, (long long)L.max_hub, h.n_seg, (long long)L.max_seg);
  if ((!small || h.n_seg > SO_SMALL) && h.n_seg <= SO_RANK) {
    const int seg_wgs = (h.n_seg + SO_SEGS - 1) / SO_SEGS, wgs = seg_wgs + (h.n_blocks + SO_THREADS - 1) / SO_THREADS;
    if (wgs > 0) {
      k_seg_rank<true><<<(unsigned)wgs, SO_THREADS, 0, s>>>(seg_key[0], ctr, seg_ord[0], items, max_items, nullptr, item_desc, seg_wgs);
      ISP_LAUNCH_CHECK();
    }
  } else if (!small || h.n_seg > SO_SMALL) {
    if (h.n_seg > 0) {  // schedule order: by first column, equal ones in order of position (stable)
      const int n_tiles = (h.n_seg + SO_TILE - 1) / SO_TILE;
      int32_t* table = (int32_t*)(base + L.so_table);
      int32_t* total = (int32_t*)(base + L.so_total);
      int bits = 1;  // the keys are columns (< n_cols)
      while (bits < 31 && ((int64_t)1 << bits) < n_cols) ++bits;
      const int n_pass = (bits + 7) / 8;
      for (int pass = 0; pass < n_pass; ++pass) {
        const int32_t* kin = seg_key[pass & 1];
        const int32_t* vin = pass == 0 ? nullptr : seg_ord[pass & 1];
        k_seg_hist<<<n_tiles, SO_TILE, 0, s>>>(kin, h.n_seg, 8 * pass, n_tiles, table);
        ISP_LAUNCH_CHECK();
        k_digit_scan<<<SO_RADIX, BS_THREADS, 0, s>>>(table, n_tiles, total);
        ISP_LAUNCH_CHECK();
        k_seg_scatter<<<n_tiles, SO_TILE, 0, s>>>(kin, vin, h.n_seg, 8 * pass, n_tiles, table, total, seg_key[(pass + 1) & 1],
                                                  seg_ord[(pass + 1) & 1]);
        ISP_LAUNCH_CHECK();
      }
      seg_order = seg_ord[n_pass & 1];
    }
    if (h.n_blocks + h.n_seg > 0) {
      k_item_desc<<<(unsigned)((h.n_blocks + h.n_seg + 255) / 256), 256, 0, s>>>(items, h.n_blocks, seg_order, h.n_seg,
                                                                               item_desc);
      ISP_LAUNCH_CHECK();
    }
  }
  out->blk_row = blk_row; out->hub_rows = hub_rows; out->hub_seg_ptr = hub_seg_ptr; out->seg_hub = seg_hub;
  out->seg_begin = seg_begin; out->hubflag = hubflag; out->seg_order = seg_order; out->item_desc = item_desc;
  out->hub_done = (unsigned*)(base + L.hub_done);
  out->partials = (float*)(base + L.partials);
  out->inv_len = (float*)(base + L.inv_len);
  return ISP_OK;
}

void fill_view(isp_view& v, int64_t n_rows, int64_t n_cols, int64_t nnz, const int64_t* indptr, const int32_t* indices,
               const float* values, const partition_out& po, const partition_params& pp) {
  v.n_rows = n_rows; v.n_cols = n_cols; v.nnz = nnz;
  v.indptr = indptr; v.indices = indices; v.values = values;
  v.blk_row = po.blk_row; v.n_blocks = po.h.n_blocks;
  v.hub_rows = po.hub_rows; v.hub_seg_ptr = po.hub_seg_ptr; v.seg_hub = po.seg_hub;
  v.seg_begin = po.seg_begin; v.seg_order = po.seg_order; v.item_desc = po.item_desc;
  v.n_hub = po.h.n_hub; v.n_seg = po.h.n_seg;
  v.hub_t = pp.hub_t; v.seg_len = pp.seg_len;
  v.partials = po.partials;
  v.hub_done = po.hub_done;
  v.inv_len = po.inv_len;
  v.n_real_rows = n_rows;
  v.piece_slot = nullptr;
}

// The packed SpMM layout of the handle's matrix (see above), into A->vp.  A->v must be filled.
isp_status build_packed(isp_csr* A, const partition_params& p1, int mid_t, char* base, const packed_layout& P,
                        size_t ws_bytes, hipStream_t s) {
  const isp_view& v = A->v;
  const int64_t n = v.n_rows, nnz = v.nnz;
  const partition_params pc = cut_params(p1, mid_t);
  partition_out cut;
  isp_status st = build_partition(n, v.n_cols, nnz, v.indptr, v.indices, pc, base, P.cut, false, -1, s, &cut);
  if (st != ISP_OK) return st;
  const int n_pc = cut.h.n_seg;
  if (cut.h.n_hub == 0) return ISP_OK;  // nothing to cut: the ordinary partition serves
  int64_t* indptr2 = (int64_t*)(base + P.indptr2);
  int32_t* indices2 = (int32_t*)(base + P.indices2);
  float* values2 = v.values ? (float*)(base + P.values2) : nullptr;
  int32_t* src_pos = (int32_t*)(base + P.src_pos);
  int32_t* len_tmp = (int32_t*)(base + P.len_tmp);
  int64_t* short_scan = (int64_t*)(base + P.scan64);
  int64_t* piece_scan = short_scan + (n + 2);
  void* scan_tmp = base + P.scan_tmp;
  k_short_len<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(v.indptr, cut.hubflag, n, len_tmp);
  ISP_LAUNCH_CHECK();
  if ((st = isp_scan_i32_to_i64(len_tmp, short_scan, n, scan_tmp, s)) != ISP_OK) return st;
  k_piece_len<<<(unsigned)((n_pc + 255) / 256), 256, 0, s>>>(v.indptr, cut.hub_rows, cut.hub_seg_ptr, cut.seg_hub,
                                                           cut.seg_begin, cut.seg_order, n_pc, len_tmp);
  ISP_LAUNCH_CHECK();
  if ((st = isp_scan_i32_to_i64(len_tmp, piece_scan, n_pc, scan_tmp, s)) != ISP_OK) return st;
  const int64_t n2 = n + n_pc;
  k_join_offsets<<<(unsigned)((n2 + 1 + 255) / 256), 256, 0, s>>>(short_scan, n, piece_scan, n_pc, indptr2);
  ISP_LAUNCH_CHECK();
  k_copy_short<<<(unsigned)((nnz + CP_TILE - 1) / CP_TILE), 256, 0, s>>>(v.indptr, v.indices, v.values, cut.hubflag, n, nnz,
                                                                       indptr2, indices2, values2, src_pos);
  ISP_LAUNCH_CHECK();
  k_copy_pieces<<<(unsigned)((n_pc + 3) / 4), 256, 0, s>>>(v.indices, v.values, cut.seg_begin, cut.seg_order, n_pc, n,
                                                         indptr2, indices2, values2, src_pos);
  ISP_LAUNCH_CHECK();
  // the derived matrix's own partition: row blocks only, none straddling the first piece row
  const partition_params pd = derived_params(p1, pc);
  const ws_layout L2 = make_layout(n2, nnz, pd, P.part2_start, false);
  if (L2.total > ws_bytes) return isp_fail(ISP_EINVAL, "internal: packed layout exceeds the workspace (%zu > %zu)", L2.total, ws_bytes);
  partition_out d2;
  if ((st = build_partition(n2, v.n_cols, nnz, indptr2, indices2, pd, base, L2, false, n, s, &d2)) != ISP_OK) return st;
  if (d2.h.n_hub != 0 || d2.h.n_seg != 0)
    return isp_fail(ISP_EINVAL, "internal: the derived matrix has %d rows above its hub threshold", d2.h.n_hub);
  isp_view& vp = A->vp;
  fill_view(vp, n2, v.n_cols, nnz, indptr2, indices2, values2, d2, pd);
  // the pieces' sums go to the cut partition's partial rows and are added by its hub tables
  vp.hub_rows = cut.hub_rows; vp.hub_seg_ptr = cut.hub_seg_ptr; vp.n_hub = cut.h.n_hub;
  vp.partials = cut.partials;
  vp.hub_done = nullptr;
  vp.inv_len = v.inv_len;
  vp.n_real_rows = n;
  vp.piece_slot = cut.seg_order;
  A->has_packed = true;
  if (n_pc > A->spmm_rows) A->spmm_rows = n_pc;
  A->packed_block_cost = pd.block_cost;
  A->packed_row_cost = pd.row_cost;
  A->packed_values_rw = values2;
  A->packed_src_pos = src_pos;
  A->info.spmm_mid_threshold = mid_t;
  A->info.spmm_cut_rows = cut.h.n_hub;
  A->info.spmm_pieces = n_pc;
  A->info.spmm_row_blocks = d2.h.n_blocks;
  return ISP_OK;
}

}  // namespace

size_t isp_partition_workspace(int64_t n_rows, int64_t n_cols, int64_t nnz, int stage_min) {
  const partition_params p1 = get_params(n_rows, nnz, isp_wave_slots(), n_cols);
  const ws_layout L = make_layout(n_rows, nnz, p1);
  const int mid_t = mid_threshold(n_rows, n_cols, nnz, p1);
  const size_t own = L.total + isp_stage::own_bytes(n_cols, nnz, L.total - L.partials, mid_t > 0, stage_min);
  if (mid_t == 0) return own;
  return make_packed_layout(n_rows, nnz, true, p1, mid_t, own).total;
}

isp_status isp_gather_values(const int32_t* pos, const float* values, int64_t nnz, float* out, hipStream_t s) {
  if (nnz >= GV_MANY_NNZ)
    k_gather_values<8><<<(unsigned)((nnz + 256 * 8 - 1) / (256 * 8)), 256, 0, s>>>(pos, values, nnz, out);
  else
    k_gather_values<1><<<(unsigned)((nnz + 255) / 256), 256, 0, s>>>(pos, values, nnz, out);
  ISP_LAUNCH_CHECK();
  return ISP_OK;
}

isp_status isp_refresh_packed_values(isp_csr* A, hipStream_t s) {
  if (!A->has_packed || !A->packed_values_rw || !A->v.values || A->v.nnz == 0) return ISP_OK;
  return isp_gather_values(A->packed_src_pos, A->v.values, A->v.nnz, A->packed_values_rw, s);
}

isp_status isp_refresh_packed_pair(isp_csr* A, hipStream_t s) {
  isp_csr* At = A->At;
  const bool shared = At && A->has_packed && At->has_packed && A->packed_values_rw && At->packed_values_rw &&
                      A->packed_src_pos == At->packed_src_pos && A->v.nnz > 0;
  if (!shared) {
    const isp_status st = isp_refresh_packed_values(A, s);
    return st != ISP_OK || !At ? st : isp_refresh_packed_values(At, s);
  }
  const int64_t nnz = A->v.nnz;
  k_gather_values_pair<<<(unsigned)((nnz + 256 * GV2_PER_THREAD - 1) / (256 * GV2_PER_THREAD)), 256, 0, s>>>(
      A->packed_src_pos, A->v.values, At->v.values, nnz, A->packed_values_rw, At->packed_values_rw);
  ISP_LAUNCH_CHECK();
  return ISP_OK;
}

isp_status isp_build_handle(int64_t n_rows, int64_t n_cols, int64_t nnz, const int64_t* indptr,
                            const int32_t* indices, const float* values, void* ws, size_t ws_bytes, bool validate,
                            const isp_tuning& tune, hipStream_t s, isp_csr** out, const int* flag, int* host_flag) {
  const partition_params pp = get_params(n_rows, nnz, isp_wave_slots(), n_cols);
  const ws_layout L = make_layout(n_rows, nnz, pp);
  const int mid_t = mid_threshold(n_rows, n_cols, nnz, pp);
  packed_layout P{};
  const size_t rows_end = L.total + isp_stage::own_bytes(n_cols, nnz, L.total - L.partials, mid_t > 0, tune.stage_min);
  size_t need = rows_end;
  if (mid_t > 0) {
    P = make_packed_layout(n_rows, nnz, values != nullptr, pp, mid_t, need);
    need = P.total;
  }
  if (ws_bytes < need) return isp_fail(ISP_EINVAL, "workspace too small: %zu < %zu bytes", ws_bytes, need);
  if (((uintptr_t)ws & 255) != 0) return isp_fail(ISP_EINVAL, "workspace must be 256-byte aligned");
  char* base = (char*)ws;
  partition_out po;
  isp_status st = build_partition(n_rows, n_cols, nnz, indptr, indices, pp, base, L, validate, -1, s, &po, flag, host_flag);
  if (st != ISP_OK) return st;

  int device = 0;
  ISP_HIP(hipGetDevice(&device));
  isp_csr* A = new (std::nothrow) isp_csr();
  if (!A) return isp_fail(ISP_ENOMEM, "host allocation of the handle failed");
  A->device = device;
  A->wave_slots = isp_wave_slots();
  A->tune = tune;
  fill_view(A->v, n_rows, n_cols, nnz, indptr, indices, values, po, pp);
  A->vp = A->v;
  A->partial_rows = L.max_seg + 1;
  A->spmm_rows = po.h.n_seg;
  A->longest_row_segs = po.h.n_hub > 0 ? (int32_t)row_segments((int64_t)po.h.max_degree, pp) : 0;
  A->has_packed = false; A->packed_values_rw = nullptr; A->packed_src_pos = nullptr;
  A->perm = nullptr; A->t_values_rw = nullptr; A->At = nullptr; A->is_transpose = false; A->mirror_aligned = false;
  A->mean_values = nullptr; A->mean_values_packed = nullptr; A->mean_values_valid = false; A->mean_values_used = false;
  A->sel_flags = nullptr; A->inv_perm = nullptr; A->inv_perm_valid = false; A->gather_bound = nullptr; A->gather_bound_valid = false;
  A->source = nullptr; A->values_gen = 0; A->source_gen = 0;
  isp_csr_info_t& I = A->info;
  const build_counters& h = po.h;
  I.n_rows = n_rows; I.n_cols = n_cols; I.nnz = nnz; I.max_degree = (int64_t)h.max_degree;
  for (int b = 0; b < 5; ++b) { I.bin_rows[b] = (int64_t)h.bin_rows[b]; I.bin_nnz[b] = (int64_t)h.bin_nnz[b]; }
  I.hub_threshold = pp.hub_t; I.segment_len = pp.seg_len; I.block_cost = pp.block_cost;
  I.n_row_blocks = h.n_blocks; I.n_hub_rows = h.n_hub; I.n_segments = h.n_seg;
  I.is_transpose = 0; I.has_cached_transpose = 0;
  I.spmm_mid_threshold = 0; I.spmm_cut_rows = 0; I.spmm_pieces = 0; I.spmm_row_blocks = 0; I.symmetric_pattern = 0;
  if (mid_t > 0 && nnz > 0) {
    st = build_packed(A, pp, mid_t, base, P, ws_bytes, s);
    if (st != ISP_OK) { delete A; return st; }
  }
  // The copies of ragged operands: among the partial rows that no operation writes, the packed layout's first; else among
  // those that a SpMM does not write (the calls on a handle follow each other).
  char* rows = base + L.partials;
  isp_stage::room rooms[3] = {
      {base + P.cut.partials + (A->has_packed ? A->info.spmm_pieces : 0) * PARTIAL_ROW, base + P.cut.total},
      {rows + isp_busy_rows(A) * PARTIAL_ROW, base + rows_end},
      {rows + (A->has_packed ? 0 : A->v.n_seg) * PARTIAL_ROW, base + rows_end}};
  isp_stage::place(A, rooms + (mid_t > 0 ? 0 : 1), mid_t > 0 ? 3 : 2);
  *out = A;
  return ISP_OK;
}
