// Stable CSR transpose, built once per graph and cached in the source handle (paper Section 3.3:
// cache-enabled backpropagation; the cached expression is read as A^T in CSR form).
//
// "Stable" = entries of one column keep their order of appearance in A, which makes the result
// unique and lets it be compared bit for bit.  It is computed as a least-significant-digit radix
// sort of the column indices (digits of up to 9 bits) that carries source position, source row and value as
// payload; every pass is a stable counting sort: per-tile digit histograms -> exclusive scan over
// (digit, tile) -> scatter with ranks taken in source order.  Integer work only, no atomics on
// anything order-dependent.
#include <new>
#include "digit_scan.h"
#include "host_slot.h"
#include "stage_rule.h"

namespace {
using namespace isp_dev;

constexpr int RS_THREADS = 256;
constexpr int RS_WAVES = RS_THREADS / ISP_WAVE;
// Keys per lane: a workgroup walks them in order, so small matrices get shorter tiles (1 M entries: 4 keys instead of 16
// spread a pass over 977 workgroups).
constexpr int RS_ROUNDS_SMALL = 4, RS_ROUNDS_LARGE = 16;
constexpr int rs_tile(int rounds) { return rounds * RS_THREADS; }  // keys per workgroup
constexpr int64_t RS_SMALL_NNZ = 4 << 20;
constexpr int RS_MAX_BITS = 9;                      // bits per digit (512 counters per wave)

// Per-tile digit histogram; table is digit-major: table[digit * n_tiles + tile].  FIRST: also finds the row that owns
// the tile's first entry (the smallest r with indptr[r + 1] > tile * RS_TILE) and clears *flag.
template <bool FIRST, int ROUNDS>
__global__ void __launch_bounds__(RS_THREADS) k_radix_hist(const int32_t* __restrict__ keys, int64_t n, int shift,
                                                           int bits, int n_tiles, int32_t* __restrict__ table,
                                                           const int64_t* __restrict__ indptr, int64_t n_rows,
                                                           int32_t* __restrict__ tile_row, int* __restrict__ flag) {
  __shared__ int hist[1 << RS_MAX_BITS];
  constexpr int RS_TILE = rs_tile(ROUNDS);
  constexpr int STRIDE = !FIRST && ROUNDS == RS_ROUNDS_SMALL ? 4 : 1;  // (keys in records)
  const int radix = 1 << bits;
  for (int i = threadIdx.x; i < radix; i += RS_THREADS) hist[i] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * RS_TILE;
  int key[ROUNDS];  // (on their way while the row is searched for)
#pragma unroll
  for (int k = 0; k < ROUNDS; ++k) {
    const int64_t q = base + k * RS_THREADS + threadIdx.x;
    key[k] = q < n ? keys[q * STRIDE] : -1;
  }
  if (FIRST) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *flag = 0;
    int64_t lo = 0, hi = n_rows - 1;  // base < nnz = indptr[n_rows], so the answer exists
    while (lo < hi) {                 // 256 probes at a time: every step is a trip to memory
      const int64_t step = (hi - lo + RS_THREADS) / RS_THREADS;
      const int64_t last = lo + (threadIdx.x + 1) * step - 1, r = last < hi ? last : hi;  // the end of this thread's part
      const int c = __syncthreads_count(indptr[r + 1] <= base);  // parts that lie before the answer
      lo += c * step;
      hi = lo + step - 1 < hi ? lo + step - 1 : hi;
    }
    if (threadIdx.x == 0) tile_row[blockIdx.x] = (int32_t)lo;
  }
#pragma unroll
  for (int k = 0; k < ROUNDS; ++k)
    if (base + k * RS_THREADS + threadIdx.x < n) atomicAdd(&hist[(key[k] >> shift) & (radix - 1)], 1);
  __syncthreads();
  for (int i = threadIdx.x; i < radix; i += RS_THREADS) table[(int64_t)i * n_tiles + blockIdx.x] = hist[i];
}

// Stable scatter of one pass; the records travel as four parallel arrays (column key, source position,
// source row, value), so the last pass leaves perm, the source rows and the values of A^T where they
// belong and nothing has to be gathered afterwards.
// Wave w of a workgroup owns the contiguous keys [tile + w * ROUNDS * 64, + ROUNDS * 64) and walks them
// 64 at a time in source order, so a key's rank among equal digits = (equal digits in earlier tiles:
// scanned table) + (in earlier waves of the tile) + (earlier rounds of this wave) + (lower lanes of this
// round).  The tile is first put in digit order in LDS and written out from there, which turns the
// scattered 4-byte stores into contiguous runs per digit.
// FIRST: the input is the CSR itself: keys = indices, source position = index, value = values (val_in), and
// the source rows are rebuilt per tile from the row offsets: every row that starts inside the tile marks its
// first position in LDS, a running maximum spreads the marks (tile_row = the row owning the tile's first entry).
// BITS: most bits a digit of this launch may have (sizes the counters in LDS).
// Short tiles (small matrices) keep a record's four numbers together, in LDS and between the passes (in the set's four
// arrays taken as one; keys_in / keys_out): a run of four equal digits is then one 64-byte piece instead of four of 16, and
// the tile is reordered once instead of four times with two barriers each (1 M entries, two passes: 24.4 + 17.3 us,
// 15.1 + 17.9 this way: the last pass writes its four arrays as before).  Long tiles fill their runs either way, and 64 KB of LDS would leave two workgroups per compute unit.
template <bool FIRST, bool LAST, bool HAS_VAL, int BITS, int ROUNDS>
__global__ void __launch_bounds__(RS_THREADS) k_radix_scatter(
    const int32_t* __restrict__ keys_in, const int32_t* __restrict__ src_in, const int32_t* __restrict__ row_in,
    const int32_t* __restrict__ val_in, const int64_t* __restrict__ indptr, int64_t n_rows,
    const int32_t* __restrict__ tile_row, int64_t n, int shift, int mask, int n_tiles,
    const int32_t* __restrict__ table_scanned, const int32_t* __restrict__ digit_total, int32_t* __restrict__ keys_out, int32_t* __restrict__ src_out,
    int32_t* __restrict__ row_out, int32_t* __restrict__ val_out) {
  constexpr int RADIX = 1 << BITS;
  constexpr int RS_ROUNDS = ROUNDS, RS_WAVE_KEYS = ROUNDS * ISP_WAVE;  // contiguous keys owned by one wave
  constexpr int RS_TILE = rs_tile(ROUNDS);
  __shared__ volatile int wave_cnt[RS_WAVES][RADIX];
  __shared__ int wave_base[RS_WAVES][RADIX];  // tile-local sorted position of each wave's first key of a digit
  __shared__ int delta[RADIX];                // output position minus tile-local position, per digit
  __shared__ int wave_tot[RS_WAVES];
  constexpr bool RECORDS = ROUNDS == RS_ROUNDS_SMALL;
  __shared__ __align__(16) int buf[RS_TILE * (RECORDS ? 4 : 1)];
  const int lane = threadIdx.x & (ISP_WAVE - 1), w = threadIdx.x / ISP_WAVE;
  for (int i = threadIdx.x; i < RS_WAVES * RADIX; i += RS_THREADS) (&wave_cnt[0][0])[i] = 0;
  const int64_t tile_base = (int64_t)blockIdx.x * RS_TILE;
  const int tile_count = (int)((n - tile_base < RS_TILE) ? n - tile_base : RS_TILE);
  const int64_t wbase = tile_base + (int64_t)w * RS_WAVE_KEYS;
  int key[RS_ROUNDS], src[RS_ROUNDS], row[RS_ROUNDS], val[RS_ROUNDS], pos[RS_ROUNDS];
#pragma unroll
  for (int r = 0; r < RS_ROUNDS; ++r) {
    const int64_t q = wbase + r * ISP_WAVE + lane;
    const bool valid = q < n;
    if constexpr (RECORDS && !FIRST) {
      const int4 rec = valid ? reinterpret_cast<const int4*>(keys_in)[q] : make_int4(0, 0, 0, 0);
      key[r] = rec.x;
      src[r] = rec.y;
      row[r] = rec.z;
      val[r] = rec.w;
    } else {
      key[r] = valid ? keys_in[q] : 0;
      src[r] = FIRST ? (int32_t)q : valid ? src_in[q] : 0;
      row[r] = !FIRST && valid ? row_in[q] : 0;
      val[r] = HAS_VAL && valid ? val_in[q] : 0;
    }
  }
  // thread t owns digits t * PER ...
  constexpr int PER = RADIX / RS_THREADS > 0 ? RADIX / RS_THREADS : 1;
  int all[PER], prior[PER];  // a digit's entries in all tiles, in the tiles before this one
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int dg = threadIdx.x * PER + k;
    const bool on = dg < RADIX && dg <= mask;
    all[k] = on ? digit_total[dg] : 0;
    prior[k] = on ? table_scanned[(int64_t)dg * n_tiles + blockIdx.x] : 0;
  }
  if (FIRST) {
    for (int i = threadIdx.x; i < RS_TILE; i += RS_THREADS) buf[i] = 0;
    __syncthreads();
    const int r_first = tile_row[blockIdx.x];
    if (threadIdx.x == 0) buf[0] = r_first;
    // rows after r_first that start inside the tile (of several empty rows sharing a start, the last one -
    // the owner of the entry there - wins)
    for (int64_t r = (int64_t)r_first + 1 + threadIdx.x; r < n_rows; r += RS_THREADS) {
      const int64_t o = indptr[r] - tile_base;
      if (o >= tile_count) break;
      atomicMax(&buf[o], (int)r);
    }
    __syncthreads();
    // running maximum over the tile: thread t owns ROUNDS consecutive positions
    int loc[RS_ROUNDS], run = 0;
#pragma unroll
    for (int k = 0; k < RS_ROUNDS; ++k) {
      const int v = buf[threadIdx.x * RS_ROUNDS + k];
      run = v > run ? v : run;
      loc[k] = run;
    }
    int inc = run;
#pragma unroll
    for (int o = 1; o < ISP_WAVE; o <<= 1) {
      const int t = __shfl_up(inc, o);
      if (lane >= o && t > inc) inc = t;
    }
    if (lane == ISP_WAVE - 1) wave_tot[w] = inc;
    __syncthreads();
    int before = __shfl_up(inc, 1);  // maximum over the lower lanes of this wave
    if (lane == 0) before = 0;
    for (int ww = 0; ww < w; ++ww) before = wave_tot[ww] > before ? wave_tot[ww] : before;
#pragma unroll
    for (int k = 0; k < RS_ROUNDS; ++k) buf[threadIdx.x * RS_ROUNDS + k] = loc[k] > before ? loc[k] : before;
  }
  __syncthreads();
  const unsigned long long lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  if (FIRST) {
#pragma unroll
    for (int r = 0; r < RS_ROUNDS; ++r) row[r] = buf[w * RS_WAVE_KEYS + r * ISP_WAVE + lane];
  }
#pragma unroll
  for (int r = 0; r < RS_ROUNDS; ++r) {
    const bool valid = wbase + r * ISP_WAVE + lane < n;
    const int dg = (key[r] >> shift) & mask;
    unsigned long long m = __ballot(valid);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
      const unsigned long long bal = __ballot((dg >> b) & 1);
      m &= ((dg >> b) & 1) ? bal : ~bal;
    }
    // m = valid lanes of this round holding the same digit as this lane
    const int before = valid ? wave_cnt[w][dg] : 0;
    pos[r] = before + __popcll(m & lt_mask);
    if (valid && (m & lt_mask) == 0) wave_cnt[w][dg] = before + __popcll(m);  // lowest lane of the group
  }
  __syncthreads();
  {  // exclusive scan of the tile's digit counts -> where each digit starts in the tile
    int cnt[PER][RS_WAVES], tot[PER], sum = 0, sum_all = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int dg = threadIdx.x * PER + k;
      tot[k] = 0;
      if (dg < RADIX) {
#pragma unroll
        for (int ww = 0; ww < RS_WAVES; ++ww) { cnt[k][ww] = wave_cnt[ww][dg]; tot[k] += cnt[k][ww]; }
      }
      sum += tot[k];
      sum_all += all[k];
    }
    int t0;
    int start = block_exclusive_scan<int>(sum, &t0);
    int before = block_exclusive_scan<int>(sum_all, &t0);  // entries with a smaller digit, in all tiles
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int dg = threadIdx.x * PER + k;
      if (dg < RADIX) {
        delta[dg] = before + prior[k] - start;
        int run = start;
#pragma unroll
        for (int ww = 0; ww < RS_WAVES; ++ww) { wave_base[ww][dg] = run; run += cnt[k][ww]; }
      }
      start += tot[k];
      before += all[k];
    }
  }
  __syncthreads();
  if constexpr (RECORDS) {
    int4* __restrict__ rec = reinterpret_cast<int4*>(buf);  // (the rows in buf have been read: barriers above)
#pragma unroll
    for (int r = 0; r < RS_ROUNDS; ++r)
      if (wbase + r * ISP_WAVE + lane < n)
        rec[wave_base[w][(key[r] >> shift) & mask] + pos[r]] = make_int4(key[r], src[r], row[r], val[r]);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < RS_ROUNDS; ++k) {
      const int i = k * RS_THREADS + threadIdx.x;
      if (i < tile_count) {
        const int4 e = rec[i];
        const int dst = delta[(e.x >> shift) & mask] + i;
        if (LAST) {
          keys_out[dst] = e.x;
          src_out[dst] = e.y;
          row_out[dst] = e.z;
          if (HAS_VAL) val_out[dst] = e.w;
        } else {
          reinterpret_cast<int4*>(keys_out)[dst] = e;
        }
      }
    }
    return;
  }
  // keys: into digit order in LDS, then out; remember both positions for the other arrays
#pragma unroll
  for (int r = 0; r < RS_ROUNDS; ++r) {
    const bool valid = wbase + r * ISP_WAVE + lane < n;
    const int dg = (key[r] >> shift) & mask;
    pos[r] = valid ? wave_base[w][dg] + pos[r] : -1;
    if (valid) buf[pos[r]] = key[r];
  }
  __syncthreads();
  int dst[RS_ROUNDS];
#pragma unroll
  for (int k = 0; k < RS_ROUNDS; ++k) {
    const int i = k * RS_THREADS + threadIdx.x;
    dst[k] = -1;
    if (i < tile_count) {
      const int kk = buf[i];
      dst[k] = delta[(kk >> shift) & mask] + i;
      keys_out[dst[k]] = kk;
    }
  }
  auto move = [&](const int (&v)[RS_ROUNDS], int32_t* __restrict__ out) {
    __syncthreads();  // everyone has read the previous array out of buf
#pragma unroll
    for (int r = 0; r < RS_ROUNDS; ++r)
      if (pos[r] >= 0) buf[pos[r]] = v[r];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < RS_ROUNDS; ++k)
      if (dst[k] >= 0) out[dst[k]] = buf[k * RS_THREADS + threadIdx.x];
  };
  move(src, src_out);
  move(row, row_out);
  if (HAS_VAL) move(val, val_out);
}

// Row offsets of A^T from the sorted column keys: an offset changes where the sorted column changes; empty columns get the
// next offset.  COMPARE (square matrices): *differs becomes 1 when A^T's offsets and indices are not, element for element,
// A's own; otherwise the pattern is symmetric with every row's columns ascending, and entry p of A^T is the mirror (j, i)
// of entry p = (i, j) of A.  (*differs is zeroed before.)
template <bool COMPARE>
__global__ void __launch_bounds__(256) k_col_offsets(const int32_t* __restrict__ skey, int64_t nnz, int64_t n_cols,
                                                     int64_t* __restrict__ t_indptr, const int32_t* __restrict__ t_indices,
                                                     const int64_t* __restrict__ indptr, const int32_t* __restrict__ indices,
                                                     int* __restrict__ differs) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  bool bad = false;
  if (q < nnz) {
    const int32_t c = skey[q];
    const int32_t prev = q > 0 ? skey[q - 1] : -1;
    if (COMPARE) bad = indices[q] != t_indices[q];
    auto offset = [&](int64_t cc, int64_t o) {
      t_indptr[cc] = o;
      if (COMPARE) bad |= indptr[cc] != o;
    };
    // (the clamp only matters for an unvalidated CSR with a column >= n_cols)
    const int64_t c_hi = c < n_cols ? (int64_t)c : n_cols - 1;
    for (int64_t cc = (int64_t)prev + 1; cc <= c_hi; ++cc) offset(cc, q);
    if (q == nnz - 1)
      for (int64_t cc = (int64_t)c + 1; cc <= n_cols; ++cc) offset(cc, nnz);
  }
  if (COMPARE && __any(bad) && (threadIdx.x & (ISP_WAVE - 1)) == 0) *differs = 1;  // (plain store of the same value from any wave)
}

// t_values[q] = values[perm[q]] for matrices whose columns are long, in blocks of rows.  In the order of q, neighbouring loads lie a row apart
// and every one fetches a line (128 B) of which it takes 4; the line's other entries belong to the next columns of the
// row, and are used when those columns are reached - after a line of every other row has passed through the L2.  Here
// each XCD walks the columns over one block of rows at a time, few enough that a line of each stays in its L2 until the
// columns it holds are done.  Workgroups go to the XCDs in turn; each takes GB_COLS columns' entries within the block
// (bound: where they begin, per block and column) and flattens them over its threads.
// 115 M entries, 233 k rows: 1076 -> 916 us (every entry still asks its L2 for a
// line); 30 M entries in 100 k uniform rows: with the packed copies of the values 650 -> 453 us.
constexpr int GB_COLS = 64;          // columns per workgroup (one lane each when they are added up)
constexpr int GB_ROWS = 16384;       // rows per block: at 128 B each half of an XCD's 4 MB of L2
constexpr int GB_XCDS = 8;
constexpr int64_t GB_MIN_NNZ = 16 << 20;  // below, the values stay in the L2s and the Infinity Cache anyway

// Blocks (a multiple of the XCDs), or 0 where a column's part would be shorter than 4 entries on average (100 M entries in
// 400 k rows, 8 to a part: 1691 -> 1403 us with the packed copies; the bounds, at most a quarter of the entries, fit the
// spare array).
int gather_blocks(int64_t n_rows, int64_t n_cols, int64_t nnz) {
  if (nnz < GB_MIN_NNZ) return 0;
  const int64_t b = ((n_rows + GB_ROWS - 1) / GB_ROWS + GB_XCDS - 1) / GB_XCDS * GB_XCDS;
  return n_cols * b * 4 <= nnz ? (int)b : 0;
}

// bound[b * n_cols + c]: first entry of column c in block b or later, for b = 0 .. n_blocks - 1.  n_chunks workgroups per
// block, all in the grid's first dimension (a matrix of 2^31 rows has 131,072 blocks, the second holds 65,535).
__global__ void __launch_bounds__(256) k_block_bounds(const int64_t* __restrict__ t_indptr,
                                                      const int32_t* __restrict__ t_indices, int64_t n_cols,
                                                      int rows_per_block, unsigned n_chunks, int32_t* __restrict__ bound) {
  const unsigned b = blockIdx.x / n_chunks;
  const int64_t c = (int64_t)(blockIdx.x % n_chunks) * blockDim.x + threadIdx.x;
  if (c >= n_cols) return;
  const int64_t row = (int64_t)b * rows_per_block;
  int64_t lo = t_indptr[c], hi = t_indptr[c + 1];
  if (b > 0) {
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      if (t_indices[mid] < row) lo = mid + 1; else hi = mid;
    }
  }
  bound[b * n_cols + c] = (int32_t)lo;
}

__global__ void __launch_bounds__(256) k_gather_blocked(const int32_t* __restrict__ perm, const float* __restrict__ values,
                                                        const int64_t* __restrict__ t_indptr,
                                                        const int32_t* __restrict__ bound, int64_t n_cols, int n_blocks,
                                                        int n_chunks, float* __restrict__ t_values) {
  __shared__ int first[GB_COLS], before[GB_COLS + 1];  // a column's first entry; entries of the columns before it
  const int xcd = blockIdx.x % GB_XCDS, turn = blockIdx.x / GB_XCDS;
  const int b = turn / n_chunks * GB_XCDS + xcd;
  const int64_t c0 = (int64_t)(turn % n_chunks) * GB_COLS;
  if (threadIdx.x < GB_COLS) {  // (the first wavefront)
    const int64_t c = c0 + threadIdx.x;
    int p = 0, len = 0;
    if (c < n_cols) {
      p = bound[b * n_cols + c];
      len = (b + 1 < n_blocks ? bound[(b + 1) * n_cols + c] : (int)t_indptr[c + 1]) - p;
    }
    const int inc = wave_inclusive_scan(len, (int)threadIdx.x);
    first[threadIdx.x] = p;
    before[threadIdx.x + 1] = inc;
    if (threadIdx.x == 0) before[0] = 0;
  }
  __syncthreads();
  const int n = before[GB_COLS];
  constexpr int U = 4;
  for (int i0 = threadIdx.x; i0 < n; i0 += 256 * U) {
    int q[U], p[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * 256 < n ? i0 + u * 256 : n - 1;
      int k = 0;  // the last column that begins at i or before it and is not empty
#pragma unroll
      for (int step = GB_COLS / 2; step > 0; step >>= 1) k += before[k + step] <= i ? step : 0;
      q[u] = first[k] + i - before[k];
      p[u] = perm[q[u]];
    }
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = values[p[u]];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i0 + u * 256 < n) t_values[q[u]] = v[u];
  }
}

// mean_values[q] = t_values[q] / len_A(t_indices[q])  (t_values absent: 1 / len), as one fp32 product with
// the reciprocal lengths the build keeps
__global__ void __launch_bounds__(256) k_mean_values(const int32_t* __restrict__ t_indices,
                                                     const float* __restrict__ t_values,
                                                     const float* __restrict__ inv_len, int64_t nnz,
                                                     float* __restrict__ mean_values) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < nnz) mean_values[q] = (t_values ? t_values[q] : 1.f) * inv_len[t_indices[q]];
}

__global__ void __launch_bounds__(256) k_inverse_perm(const int32_t* __restrict__ perm, int64_t nnz,
                                                      int32_t* __restrict__ inv_perm) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < nnz) inv_perm[perm[q]] = (int32_t)q;
}

__global__ void __launch_bounds__(256) k_fill_i64(int64_t* __restrict__ a, int64_t n, int64_t v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] = v;
}

struct t_layout {
  size_t t_indptr, t_indices, perm, t_values, set[2][4], tile_row, table, digit_total, flag, part, total;
  int64_t n_tiles;
  bool small;  // RS_ROUNDS_SMALL keys per lane
};

t_layout make_layout(const isp_csr* A) {
  const int64_t n_rows = A->v.n_rows, n_cols = A->v.n_cols, nnz = A->v.nnz;
  const bool has_values = A->v.values != nullptr;
  t_layout L;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += isp_align(bytes); return o; };
  L.small = nnz <= RS_SMALL_NNZ;
  const int tile = rs_tile(L.small ? RS_ROUNDS_SMALL : RS_ROUNDS_LARGE);
  L.n_tiles = (nnz + tile - 1) / tile;
  const size_t e = (size_t)(nnz + 1) * 4;
  L.t_indptr = take((size_t)(n_cols + 1) * 8);
  L.t_indices = take(e);
  L.perm = take(e);
  L.t_values = take(has_values ? e : 0);
  // two sets of record arrays (key, source position, source row, value) that the passes alternate between (small
  // matrices: of records of the four)
  for (int k = 0; k < 2; ++k)
    for (int a = 0; a < 4; ++a) L.set[k][a] = take(a == 3 && !has_values && !L.small ? 0 : e);
  L.tile_row = take((size_t)(L.n_tiles + 1) * 4);
  L.table = take((size_t)(((int64_t)L.n_tiles << RS_MAX_BITS) + 1) * 4);
  L.digit_total = take((size_t)(1 << RS_MAX_BITS) * 4);
  L.flag = take(4);
  L.part = take(isp_partition_workspace(n_cols, n_rows, nnz, A->tune.stage_min));  // (A^T: n_cols rows, n_rows columns)
  L.total = off;
  return L;
}

// Bytes share_handle takes of the transpose's workspace (besides the copy of a ragged operand).
size_t share_bytes(const isp_csr* A) {
  return isp_align((size_t)isp_shared_rows(A) * ISP_PARTIAL_TILE * sizeof(float)) +
         (A->has_packed ? isp_align((size_t)A->v.nnz * sizeof(float)) : 0);
}

// The transpose's handle when its offsets and indices equal A's: A's partition tables and packed layout, which are
// only read, serve both; values and scratch are its own (scratch: the partial rows of either partition in front, then the
// packed values, share_bytes in all; the copy of a ragged operand behind them, or among the partial rows that are not
// written; scratch_end: of what the matrix asks for, so that more workspace changes nothing).
isp_status share_handle(const isp_csr* A, const int64_t* t_indptr, const int32_t* t_indices, float* t_values,
                        char* scratch, char* scratch_end, hipStream_t s, isp_csr** out) {
  isp_csr* At = new (std::nothrow) isp_csr(*A);
  if (!At) return isp_fail(ISP_ENOMEM, "host allocation of the handle failed");
  At->At = nullptr;
  At->v.indptr = t_indptr;
  At->v.indices = t_indices;
  At->v.values = t_values;
  At->v.partials = (float*)scratch;
  At->v.hub_done = nullptr;  // (this workspace has no counters of its own: hub rows are left to the fix-up launch)
  At->partial_rows = isp_shared_rows(A);
  const size_t row = ISP_PARTIAL_TILE * sizeof(float);
  char* rows_end = scratch + isp_align((size_t)At->partial_rows * row);
  char* behind = rows_end;
  if (A->has_packed) {
    At->packed_values_rw = t_values ? (float*)behind : nullptr;
    At->vp.values = At->packed_values_rw;
    At->vp.partials = At->v.partials;
    behind += isp_align((size_t)A->v.nnz * sizeof(float));
  } else {
    At->vp = At->v;
  }
  const int64_t busy = isp_busy_rows(At);
  isp_stage::room rooms[3] = {{behind, scratch_end},
                              {scratch + (size_t)(busy > At->spmm_rows ? busy : At->spmm_rows) * row, rows_end},
                              {scratch + (size_t)At->spmm_rows * row, rows_end}};
  isp_stage::place(At, rooms, 3);
  const isp_status st = isp_refresh_packed_values(At, s);
  if (st != ISP_OK) { delete At; return st; }
  *out = At;
  return ISP_OK;
}

}  // namespace

size_t isp_transpose_workspace_bytes(const isp_csr* A) {
  return make_layout(A).total;
}

isp_status isp_transpose_build(isp_csr* A, void* ws, size_t ws_bytes, hipStream_t s) {
  const isp_view& v = A->v;
  const int64_t nnz = v.nnz, n_cols = v.n_cols, n_rows = v.n_rows;
  const bool has_values = v.values != nullptr;
  const t_layout L = make_layout(A);
  if (!ws) return isp_fail(ISP_EINVAL, "transpose workspace is NULL");
  if (ws_bytes < L.total) return isp_fail(ISP_EINVAL, "transpose workspace too small: %zu < %zu bytes", ws_bytes, L.total);
  if (((uintptr_t)ws & 255) != 0) return isp_fail(ISP_EINVAL, "workspace must be 256-byte aligned");
  char* base = (char*)ws;
  int64_t* t_indptr = (int64_t*)(base + L.t_indptr);
  int32_t* t_indices = (int32_t*)(base + L.t_indices);
  int32_t* perm = (int32_t*)(base + L.perm);
  float* t_values = has_values ? (float*)(base + L.t_values) : nullptr;
  int32_t* tile_row = (int32_t*)(base + L.tile_row);
  int32_t* table = (int32_t*)(base + L.table);
  int32_t* digit_total = (int32_t*)(base + L.digit_total);
  int* differs = (int*)(base + L.flag);

  if (nnz == 0) {
    k_fill_i64<<<(unsigned)((n_cols + 1 + 255) / 256), 256, 0, s>>>(t_indptr, n_cols + 1, 0);
    ISP_LAUNCH_CHECK();
  } else {
    int bits = 1;
    while (bits < 31 && ((int64_t)1 << bits) < n_cols) ++bits;
    // Digits of at most 8 bits, on small matrices 9 where that saves a pass (17 and 18 bits; large ones write shorter
    // runs per digit then: 115 M entries, 18 bits, 6.9 ms in three passes, 7.6 in two; 5-, 6- and 7-bit digits
    // measured slower too).
    const int n_pass = L.small && (bits + 8) / 9 < (bits + 7) / 8 ? (bits + 8) / 9 : (bits + 7) / 8;
    const int n_tiles = (int)L.n_tiles;
    const int32_t* in[4] = {v.indices, nullptr, nullptr, (const int32_t*)v.values};
    for (int pass = 0; pass < n_pass; ++pass) {
      // digits of about equal width: pass p takes bits [p * bits / n_pass, (p + 1) * bits / n_pass)
      const int shift = pass * bits / n_pass;
      const int width = (pass + 1) * bits / n_pass - shift;
      const int mask = (1 << width) - 1;
#define ISP_GO(F, R)                                                                                                 \
  k_radix_hist<F, R><<<n_tiles, RS_THREADS, 0, s>>>(in[0], nnz, shift, width, n_tiles, table, v.indptr, n_rows, tile_row, differs)
      if (L.small) { if (pass == 0) ISP_GO(true, RS_ROUNDS_SMALL); else ISP_GO(false, RS_ROUNDS_SMALL); }
      else { if (pass == 0) ISP_GO(true, RS_ROUNDS_LARGE); else ISP_GO(false, RS_ROUNDS_LARGE); }
#undef ISP_GO
      ISP_LAUNCH_CHECK();
      k_digit_scan<<<1 << width, RS_THREADS, 0, s>>>(table, n_tiles, digit_total);
      ISP_LAUNCH_CHECK();
      int32_t* out[4];
      for (int a = 0; a < 4; ++a) out[a] = (int32_t*)(base + L.set[pass & 1][a]);
      if (pass == n_pass - 1) {  // the last pass writes A^T's arrays; its keys still go to the set (for the offsets)
        out[1] = perm;
        out[2] = t_indices;
        out[3] = (int32_t*)t_values;
      }
#define ISP_GO(F, LA, HV, B, R)                                                                                      \
  k_radix_scatter<F, LA, HV, B, R><<<n_tiles, RS_THREADS, 0, s>>>(in[0], in[1], in[2], in[3], v.indptr, n_rows, tile_row, nnz, \
                                                               shift, mask, n_tiles, table, digit_total, out[0], out[1], out[2], out[3])
#define ISP_GO2(F, LA, HV)                                                                                           \
  do {                                                                                                               \
    if (width > 8) ISP_GO(F, LA, HV, 9, RS_ROUNDS_SMALL); else ISP_GO(F, LA, HV, 8, RS_ROUNDS_SMALL);                     \
  } while (0)
#define ISP_GO3(F, LA) do { if (has_values) ISP_GO2(F, LA, true); else ISP_GO2(F, LA, false); } while (0)
#define ISP_GO4(F) do { if (has_values) ISP_GO(F, true, true, 8, RS_ROUNDS_LARGE); else ISP_GO(F, true, false, 8, RS_ROUNDS_LARGE); } while (0)
      const bool first = pass == 0, last = pass == n_pass - 1;
      if (!L.small) { if (first) ISP_GO4(true); else ISP_GO4(false); }  // (four arrays in and out in every pass)
      else if (first && last) ISP_GO3(true, true);
      else if (first) ISP_GO3(true, false);
      else if (last) ISP_GO3(false, true);
      else ISP_GO3(false, false);
#undef ISP_GO4
#undef ISP_GO3
#undef ISP_GO2
#undef ISP_GO
      ISP_LAUNCH_CHECK();
      for (int a = 0; a < 4; ++a) in[a] = out[a];
    }
    // (and is the pattern symmetric?  The first histogram has cleared the flag.)
#define ISP_GO(C)                                                                                                    \
  k_col_offsets<C><<<(unsigned)((nnz + 255) / 256), 256, 0, s>>>(in[0], nnz, n_cols, t_indptr, t_indices, v.indptr, v.indices, \
                                                                 differs)
    if (n_rows == n_cols) ISP_GO(true); else ISP_GO(false);
#undef ISP_GO
    ISP_LAUNCH_CHECK();
  }
  const bool square = n_rows == n_cols && nnz > 0;
  isp_csr* At = nullptr;
  isp_status st;
  int h_differs = 1;
  host_slot slot;
  int* host_flag = square ? (int*)slot.get() : nullptr;
  const bool ask_first = square && nnz > RS_SMALL_NNZ;
  if (ask_first) {
    // A^T of a symmetric pattern has A's partitions: on a large matrix a round trip to the host is nothing beside
    // building them again (115 M entries: 2.5 of 6.6 ms).
    ISP_HIP(hipMemcpyAsync(host_flag ? host_flag : &h_differs, differs, sizeof(int), hipMemcpyDeviceToHost, s));
    ISP_HIP(hipStreamSynchronize(s));
    if (host_flag) h_differs = *host_flag;
  }
  if (ask_first && h_differs == 0 && share_bytes(A) <= L.total - L.part) {
    if ((st = share_handle(A, t_indptr, t_indices, t_values, base + L.part, base + L.total, s, &At)) != ISP_OK) return st;
  } else {
    // (on a small one the flag comes to the host with the partition's counters)
    int* with_counters = ask_first ? nullptr : host_flag;
    st = isp_build_handle(n_cols, n_rows, nnz, t_indptr, t_indices, t_values, base + L.part, ws_bytes - L.part, false, A->tune, s,
                          &At, differs, with_counters);
    if (st != ISP_OK) return st;
    if (with_counters) {
      h_differs = *with_counters;
    } else if (square && !ask_first) {
      ISP_HIP(hipMemcpyAsync(&h_differs, differs, sizeof(int), hipMemcpyDeviceToHost, s));
      ISP_HIP(hipStreamSynchronize(s));
    }
  }
  A->mirror_aligned = At->mirror_aligned = (h_differs == 0);
  A->info.symmetric_pattern = At->info.symmetric_pattern = A->mirror_aligned ? 1 : 0;
  At->perm = perm;
  At->t_values_rw = t_values;
  // the record arrays of the sort are free from here on; one of them later holds the mean reduction's values
  At->mean_values = (float*)(base + L.set[0][1]);
  At->mean_values_packed = At->has_packed ? (float*)(base + L.set[1][2]) : nullptr;
  At->mean_values_valid = false;
  At->mean_values_used = false;
  At->sel_flags = (uint8_t*)(base + L.set[1][1]);
  At->inv_perm = (int32_t*)(base + L.set[0][2]);
  At->inv_perm_valid = false;
  At->gather_bound = has_values && gather_blocks(n_rows, n_cols, nnz) ? (int32_t*)(base + L.set[0][0]) : nullptr;
  At->gather_bound_valid = false;
  At->is_transpose = true;
  At->info.is_transpose = 1;
  A->At = At;
  A->info.has_cached_transpose = 1;
  return ISP_OK;
}

namespace {
// While s is being captured into a HIP graph the kernels enqueued here run only when the graph is replayed:
// the fill is then part of every replay and the cache is not marked filled.
bool stream_is_capturing(hipStream_t s) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &st) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return st == hipStreamCaptureStatusActive;
}

}  // namespace

// (and, where A^T has the packed SpMM layout, the same values in the order of that layout's entries)
static isp_status fill_mean_values(isp_csr* A, hipStream_t s) {
  isp_csr* At = A->At;
  const unsigned grid = (unsigned)((A->v.nnz + 255) / 256);
  k_mean_values<<<grid, 256, 0, s>>>(At->v.indices, At->v.values, A->v.inv_len, A->v.nnz, At->mean_values);
  ISP_LAUNCH_CHECK();
  if (At->mean_values_packed) {
    return isp_gather_values(At->packed_src_pos, At->mean_values, A->v.nnz, At->mean_values_packed, s);
  }
  return ISP_OK;
}

isp_status isp_transpose_mean_values(isp_csr* A, hipStream_t s, const float** out, const float** out_packed) {
  isp_csr* At = A->At;
  if (!At || !At->mean_values) return isp_fail(ISP_EINVAL, "no cached transpose");
  if (!At->mean_values_valid && A->v.nnz > 0) {
    isp_status st = fill_mean_values(A, s);
    if (st != ISP_OK) return st;
    At->mean_values_valid = !stream_is_capturing(s);
  }
  At->mean_values_used = true;
  *out = At->mean_values;
  *out_packed = At->mean_values_packed;
  return ISP_OK;
}

isp_status isp_transpose_inverse_perm(isp_csr* A, hipStream_t s, const int32_t** out) {
  isp_csr* At = A->At;
  if (!At || !At->inv_perm) return isp_fail(ISP_EINVAL, "no cached transpose");
  if (!At->inv_perm_valid && A->v.nnz > 0) {
    k_inverse_perm<<<(unsigned)((A->v.nnz + 255) / 256), 256, 0, s>>>(At->perm, A->v.nnz, At->inv_perm);
    ISP_LAUNCH_CHECK();
    At->inv_perm_valid = !stream_is_capturing(s);
  }
  *out = At->inv_perm;
  return ISP_OK;
}

// Everything derived from A's values is brought up to date on s itself, in stream order: a call recorded into a
// HIP graph refreshes on every replay, and a graph that was captured while the mean reduction's values were
// valid (and therefore holds no pass that computes them) reads refreshed ones after an eager call.
isp_status isp_transpose_refresh_values(isp_csr* A, hipStream_t s) {
  isp_csr* At = A->At;
  if (!At || !A->v.values || !At->t_values_rw || A->v.nnz == 0) return ISP_OK;
  if (At->gather_bound) {
    const int n_blocks = gather_blocks(A->v.n_rows, A->v.n_cols, A->v.nnz);
    const int n_chunks = (int)((A->v.n_cols + GB_COLS - 1) / GB_COLS);
    if (!At->gather_bound_valid) {  // (115 M entries, 233 k columns: 216 us once)
      const unsigned chunks = (unsigned)((A->v.n_cols + 255) / 256);  // (n_cols * n_blocks <= nnz / 4: gather_blocks)
      k_block_bounds<<<chunks * (unsigned)n_blocks, 256, 0, s>>>(At->v.indptr, At->v.indices, A->v.n_cols,
                                                                 (int)((A->v.n_rows + n_blocks - 1) / n_blocks), chunks,
                                                                 At->gather_bound);
      ISP_LAUNCH_CHECK();
      At->gather_bound_valid = !stream_is_capturing(s);
    }
    k_gather_blocked<<<(unsigned)(n_chunks * n_blocks), 256, 0, s>>>(At->perm, A->v.values, At->v.indptr, At->gather_bound,
                                                                   A->v.n_cols, n_blocks, n_chunks, At->t_values_rw);
    ISP_LAUNCH_CHECK();
  } else {
    const isp_status st = isp_gather_values(At->perm, A->v.values, A->v.nnz, At->t_values_rw, s);
    if (st != ISP_OK) return st;
  }
  if (At->mean_values_used) {  // a mean backward has run (or was captured): its values follow at once
    isp_status st = fill_mean_values(A, s);
    if (st != ISP_OK) return st;
    // (valid stays as it is: during a capture the refill runs with the replays, like the fill itself)
  }
  return ISP_OK;
}
