// CSR transpose of A on the device (the A^T of the products A^T y, of the
// assembly and of the adjoint).
//
// The entries are sorted by column with a least-significant-digit radix sort
// on the column index (digits of up to 11 bits, of equal width over as few
// passes as the column count needs), carrying each entry's index in A as its
// value.  Every pass is a stable counting sort, so inside a column the
// entries keep A's order, that is ascending rows.  A pass:
//   1. k_digit_hist: per tile of RS_TILE keys a digit histogram, stored
//      digit-major (hist[digit * ntiles + tile]);
//   2. an exclusive scan of that array: the first output position of every
//      (digit, tile) pair;
//   3. k_digit_scatter: each tile ranks its keys among equal digits in input
//      order, orders itself in LDS and writes keys and values in runs.
// The row pointer of A^T comes from the sorted columns.  The row and the
// value of each entry travel through the passes with it where the work space
// has room (carry); else they are gathered at the end (k_rows_of).
//
// What bounds it: the bytes of the passes.  1.9e7 entries, 1e6 columns, random
// row order: 3.05 ms -> 0.95 ms of kernels.  Before, rows by binary search
// over the whole row pointer and a gather of the values took 1.44 ms, three
// 8-bit passes written entry by entry 0.97, column counts by global atomics
// 0.51; with the present passes a gather of rows and values (one line of 64
// entries searched per entry) still took 0.66 ms, while carrying them adds 0.40.
#include <mutex>
#include <string>

#include "kernels.hpp"

namespace lsq2l {

constexpr int RS_THREADS = 512;                 // threads of a sort workgroup
constexpr int RS_WAVES = RS_THREADS / 64;
constexpr int RS_ITEMS = 16;                    // keys per thread and tile
constexpr int RS_TILE = RS_THREADS * RS_ITEMS;  // keys per tile
// Widest digit: 2,048 counters of 16 bits per wave, with the 8,192 staged
// words and one table of the digits, are 72 KB of LDS, two workgroups per CU.
// Columns up to 2^22 then take two passes.
constexpr int RS_BITS = 11;
constexpr int RS_BINS = 1 << RS_BITS;
constexpr int RS_NARROW = 8;                    // digit width where the work space is short
constexpr int ROWTAB_SHIFT = 6;                 // entries per line of the row table (log2)
constexpr int SCAN_THREADS = 256, SCAN_ITEMS = 8, SCAN_TILE = SCAN_THREADS * SCAN_ITEMS;

// ---------------------------------------------------------------------------
// exclusive scan of int32 counts (in place), three phases
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(SCAN_THREADS)
k_scan_tiles(int64_t n, const int32_t* __restrict__ in, int32_t* __restrict__ tile_sum) {
  __shared__ int sh[4];
  const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
  int s = 0;
#pragma unroll
  for (int q = 0; q < SCAN_ITEMS; ++q)
    if (base + q < n) s += in[base + q];
  int tot = 0;
  (void)block_excl_scan_256(s, sh, &tot);
  if (threadIdx.x == 0) tile_sum[blockIdx.x] = tot;
}

// exclusive scan of the tile sums by one workgroup, in chunks of 256
__global__ void __launch_bounds__(SCAN_THREADS)
k_scan_sums(int32_t ntiles, int32_t* __restrict__ tile_sum) {
  __shared__ int sh[4];
  int carry = 0;
  for (int32_t b0 = 0; b0 < ntiles; b0 += SCAN_THREADS) {
    const int32_t t = b0 + threadIdx.x;
    const int v = t < ntiles ? tile_sum[t] : 0;
    int tot = 0;
    const int ex = block_excl_scan_256(v, sh, &tot);
    if (t < ntiles) tile_sum[t] = carry + ex;
    carry += tot;
  }
}

__global__ void __launch_bounds__(SCAN_THREADS)
k_scan_apply(int64_t n, int32_t* __restrict__ v, const int32_t* __restrict__ tile_sum) {
  __shared__ int sh[4];
  const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
  int x[SCAN_ITEMS];
  int s = 0;
#pragma unroll
  for (int q = 0; q < SCAN_ITEMS; ++q) {
    x[q] = base + q < n ? v[base + q] : 0;
    s += x[q];
  }
  int tot = 0;
  int run = tile_sum[blockIdx.x] + block_excl_scan_256(s, sh, &tot);
#pragma unroll
  for (int q = 0; q < SCAN_ITEMS; ++q)
    if (base + q < n) {
      v[base + q] = run;
      run += x[q];
    }
}

static int64_t scan_tiles(int64_t n) { return (n + SCAN_TILE - 1) / SCAN_TILE; }

// in-place exclusive scan of v[0..n); work: scan_tiles(n) int32
static void exclusive_scan(hipStream_t st, int64_t n, int32_t* v, int32_t* work) {
  if (n == 0) return;
  const unsigned nt = (unsigned)scan_tiles(n);
  k_scan_tiles<<<nt, SCAN_THREADS, 0, st>>>(n, v, work);
  k_scan_sums<<<1, SCAN_THREADS, 0, st>>>((int32_t)nt, work);
  k_scan_apply<<<nt, SCAN_THREADS, 0, st>>>(n, v, work);
}

int64_t scan_work_len(int64_t n) { return scan_tiles(n) + 1; }
void launch_exclusive_scan(hipStream_t st, int64_t n, int32_t* v, int32_t* work) {
  exclusive_scan(st, n, v, work);
}

// ---------------------------------------------------------------------------
// radix sort passes
// ---------------------------------------------------------------------------
// tab[b] = the row of A holding entry 64 b (the last one: m - 1)
__global__ void k_row_table(int64_t nnz, int32_t m, const int32_t* __restrict__ rowptr, int64_t nb,
                            int32_t* __restrict__ tab) {
  const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (b > nb) return;
  const int64_t e = b << ROWTAB_SHIFT;
  int32_t lo = 0, hi = m - 1;             // largest r with rowptr[r] <= e
  if (e >= nnz) lo = hi;
  while (lo < hi) {
    const int32_t mid = (int32_t)(((int64_t)lo + hi + 1) >> 1);
    if (rowptr[mid] <= e) lo = mid; else hi = mid - 1;
  }
  tab[b] = lo;
}

// row of entry e: the last one starting at or before e among the rows its
// table line spans
__device__ inline int32_t row_of_entry(int32_t e, const int32_t* __restrict__ rowptr,
                                       const int32_t* __restrict__ tab) {
  int32_t lo = tab[e >> ROWTAB_SHIFT], hi = tab[(e >> ROWTAB_SHIFT) + 1];
  while (lo < hi) {
    const int32_t mid = (int32_t)(((int64_t)lo + hi + 1) >> 1);
    if (rowptr[mid] <= e) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// What a pass moves beside the keys: the entry's index in A (perm; null in:
// the first pass, whose entries are in A's order), and with carry its row
// (null in: from A's row pointer and its table) and its value (may be null)
struct SortCarry {
  const int32_t* perm;
  const int32_t* row;
  const double* val;
  int32_t* operm;
  int32_t* orow;
  double* oval;
};

// key of entry k in the first pass is colind[k] and its value k; later passes
// read the previous pass's output
__global__ void __launch_bounds__(RS_THREADS)
k_digit_hist(int64_t nnz, const int32_t* __restrict__ keys, int shift, int nbits,
             int32_t* __restrict__ hist, int32_t ntiles) {
  __shared__ int cnt[RS_BINS];
  const int bins = 1 << nbits;
  for (int b = threadIdx.x; b < bins; b += RS_THREADS) cnt[b] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * RS_TILE;
#pragma unroll
  for (int q = 0; q < RS_ITEMS; ++q) {
    const int64_t k = base + (int64_t)q * RS_THREADS + threadIdx.x;
    if (k < nnz) atomicAdd(&cnt[(keys[k] >> shift) & (bins - 1)], 1);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < bins; b += RS_THREADS) hist[(int64_t)b * ntiles + blockIdx.x] = cnt[b];
}

// Tile of workgroup b: workgroup b runs on XCD b % 8, and the tiles of one
// XCD are neighbours, so that the runs which neighbouring tiles write next to
// each other for the same digit meet in one L2 and leave it as whole lines
// (a pass with rows and values carried: 0.41 -> 0.36 ms, 1.9e7 entries).
__device__ inline int32_t tile_of_block(int32_t b, int32_t ntiles) {
  const int32_t per = ntiles / 8, rest = ntiles % 8, x = b % 8;
  return x * per + min(x, rest) + b / 8;
}

// Stable scatter of one tile.  Wave w owns the keys w * 1024 .. of the tile
// and ranks them by itself, 64 at a time: the lanes holding the same digit
// (nbits ballots) take consecutive ranks after the wave's count of that digit
// so far, kept in LDS, so the ranking needs no workgroup barrier.  The counts
// of the waves are then added in wave order and the digits scanned, which
// gives every key its place in the tile's sorted order; keys and values are
// put there in LDS, one 32-bit word per entry at a time (a double goes as two
// words, which keeps the LDS at two workgroups per CU), and leave in that
// order, equal digits as one run.  Writing
// every entry straight to its output position (the form with 256 digits and
// four barriers per 256 keys) took 0.23 - 0.40 ms per pass of 1.9e7 entries;
// this one takes 0.16 ms with two passes instead of three, 0.36 ms with the
// rows and values carried.
__global__ void __launch_bounds__(RS_THREADS)
k_digit_scatter(int64_t nnz, const int32_t* __restrict__ keys, SortCarry C, int shift, int nbits,
                const int32_t* __restrict__ hist, int32_t ntiles, int32_t* __restrict__ okeys,
                const int32_t* __restrict__ rowptr, const int32_t* __restrict__ tab) {
  __shared__ uint16_t wcnt[RS_WAVES][RS_BINS];   // per wave: count, then its first place in the tile
  __shared__ int out0[RS_BINS];                  // output position of place 0, by digit
  __shared__ int stage[RS_TILE];
  __shared__ int sh[RS_WAVES];
  const int tid = threadIdx.x, lane = tid % 64, w = tid / 64;
  const int bins = 1 << nbits;
  const int32_t tile = tile_of_block(blockIdx.x, ntiles);
  const int64_t base = (int64_t)tile * RS_TILE;
  const int count = (int)min((int64_t)RS_TILE, nnz - base);
  int key[RS_ITEMS], place[RS_ITEMS];
#pragma unroll
  for (int q = 0; q < RS_ITEMS; ++q) {
    const int i = w * (64 * RS_ITEMS) + q * 64 + lane;
    key[q] = i < count ? keys[base + i] : 0;
  }
  for (int b = lane; b < bins; b += 64) wcnt[w][b] = 0;
  wave_sync();
  const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
  for (int q = 0; q < RS_ITEMS; ++q) {
    const int i = w * (64 * RS_ITEMS) + q * 64 + lane;
    const int dg = (key[q] >> shift) & (bins - 1);
    unsigned long long peers = __ballot(i < count);
    for (int b = 0; b < nbits; ++b) {
      const unsigned long long m = __ballot((dg >> b) & 1);
      peers &= ((dg >> b) & 1) ? m : ~m;
    }
    const int rank = __popcll(peers & below);
    const int seen = wcnt[w][dg];
    wave_sync();
    if (i < count && rank == 0) wcnt[w][dg] = (uint16_t)(seen + __popcll(peers));
    wave_sync();
    place[q] = seen + rank;
  }
  __syncthreads();
  // digits 4 t .. 4 t + 3 of thread t: counts over the waves, and the scan
  constexpr int BT = RS_BINS / RS_THREADS;
  int sum = 0;
#pragma unroll
  for (int u = 0; u < BT; ++u) {
    const int b = tid * BT + u;
    if (b < bins)
      for (int p = 0; p < RS_WAVES; ++p) sum += wcnt[p][b];
  }
  int x = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) sh[w] = x;
  __syncthreads();
  int at = x - sum;
  for (int p = 0; p < w; ++p) at += sh[p];
#pragma unroll
  for (int u = 0; u < BT; ++u) {
    const int b = tid * BT + u;
    if (b < bins) {
      out0[b] = hist[(int64_t)b * ntiles + tile] - at;
      for (int p = 0; p < RS_WAVES; ++p) {
        const int c = wcnt[p][b];
        wcnt[p][b] = (uint16_t)at;
        at += c;
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < RS_ITEMS; ++q) {
    const int i = w * (64 * RS_ITEMS) + q * 64 + lane;
    const int dg = (key[q] >> shift) & (bins - 1);
    place[q] += wcnt[w][dg];
    if (i < count) stage[place[q]] = key[q];
  }
  __syncthreads();
  int pos[RS_ITEMS];
#pragma unroll
  for (int q = 0; q < RS_ITEMS; ++q) {
    const int i = q * RS_THREADS + tid;
    if (i < count) {
      const int k = stage[i];
      pos[q] = out0[(k >> shift) & (bins - 1)] + i;
      okeys[pos[q]] = k;
    }
  }
  // one word per entry from input order (word(q, k): entry k of the pass, item
  // q of the thread) to sorted order (put(p, w): output position p)
  auto through = [&](auto word, auto put) {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < RS_ITEMS; ++q) {
      const int i = w * (64 * RS_ITEMS) + q * 64 + lane;
      if (i < count) stage[place[q]] = word(q, base + i);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < RS_ITEMS; ++q) {
      const int i = q * RS_THREADS + tid;
      if (i < count) put(q, stage[i]);
    }
  };
  through([&](int, int64_t k) { return C.perm ? C.perm[k] : (int32_t)k; },
          [&](int q, int32_t v) { C.operm[pos[q]] = v; });
  if (C.orow)
    through([&](int, int64_t k) { return C.row ? C.row[k] : row_of_entry((int32_t)k, rowptr, tab); },
            [&](int q, int32_t v) { C.orow[pos[q]] = v; });
  if (C.oval) {
    double v[RS_ITEMS];
    int lo[RS_ITEMS];
    through([&](int q, int64_t k) { v[q] = C.val[k]; return __double2loint(v[q]); },
            [&](int q, int32_t x) { lo[q] = x; });
    through([&](int q, int64_t) { return __double2hiint(v[q]); },
            [&](int q, int32_t x) { C.oval[pos[q]] = __hiloint2double(x, lo[q]); });
  }
}

// trowptr[c] = number of sorted columns below c, c = 0 .. n
__global__ void k_col_starts(int64_t nnz, const int32_t* __restrict__ sorted, int32_t n,
                             int32_t* __restrict__ trowptr) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c > n) return;
  int64_t lo = 0, hi = nnz;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (sorted[mid] < c) lo = mid + 1; else hi = mid;
  }
  trowptr[c] = (int32_t)lo;
}

__global__ void k_zero_fill_i32(int64_t n, int32_t v, int32_t* __restrict__ out) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) out[k] = v;
}

// trow[k] = the row of A holding entry tperm[k]; tvals[k] = vals[tperm[k]].
// Bound by the gathers: four entries per thread keep their chains of loads in
// flight together.
constexpr int ROWS_U = 4;
__global__ void __launch_bounds__(256)
k_rows_of(int64_t nnz, const int32_t* __restrict__ rowptr, const int32_t* __restrict__ tab,
          const int32_t* __restrict__ tperm, const double* __restrict__ vals,
          int32_t* __restrict__ trow, double* __restrict__ tvals) {
  const int64_t k0 = (int64_t)blockIdx.x * (256 * ROWS_U) + threadIdx.x;
  int32_t e[ROWS_U];
  double v[ROWS_U];
#pragma unroll
  for (int u = 0; u < ROWS_U; ++u) e[u] = k0 + 256 * u < nnz ? tperm[k0 + 256 * u] : 0;
#pragma unroll
  for (int u = 0; u < ROWS_U; ++u)
    if (tvals) v[u] = vals[e[u]];
#pragma unroll
  for (int u = 0; u < ROWS_U; ++u) {
    const int32_t r = row_of_entry(e[u], rowptr, tab);
    const int64_t k = k0 + 256 * u;
    if (k < nnz) {
      trow[k] = r;
      if (tvals) tvals[k] = v[u];
    }
  }
}

static int key_bits(int32_t n) {
  int b = 1;
  while (b < 31 && ((int64_t)1 << b) < n) ++b;
  return b;
}

static int passes_for(int32_t n, int width) { return (key_bits(n) + width - 1) / width; }
static int digit_bits(int32_t n, int width) {
  const int P = passes_for(n, width);
  return (key_bits(n) + P - 1) / P;
}

static int64_t hist_words(int64_t nnz, int32_t n, int width) {
  return ((nnz + RS_TILE - 1) / RS_TILE) << digit_bits(n, width);
}
static int64_t tab_words(int64_t nnz) { return (nnz >> ROWTAB_SHIFT) + 2; }
static int64_t even(int64_t x) { return (x + 1) / 2 * 2; }

// Work space: histogram, its scan, the row table; ping-pong keys and entry
// indices where there is more than one pass; with carry also rows, values and
// the sorted keys (the output row array holds rows then).
static size_t temp_bytes_for(int64_t nnz, int32_t n, int width, bool carry) {
  const int64_t hist = hist_words(nnz, n, width);
  const int64_t pp = passes_for(n, width) >= 2 ? 2 * nnz : 0;
  const int64_t words = even(hist + scan_tiles(hist) + 1 + tab_words(nnz) + pp) + (carry ? 4 * nnz : 0);
  return (size_t)((words * 4 + 255) / 256 * 256);
}

size_t transpose_temp_bytes(int64_t nnz, int32_t n) { return temp_bytes_for(nnz, n, RS_BITS, true); }
size_t transpose_temp_least(int64_t nnz, int32_t n) { return temp_bytes_for(nnz, n, RS_NARROW, false); }

// With less than transpose_temp_bytes, rows and values are gathered after the
// sort, and with less room still the digits are RS_NARROW bits wide (an
// eighth of the histogram, more passes).
hipError_t launch_transpose(hipStream_t st, int32_t m, int32_t n, int64_t nnz, const int32_t* rowptr,
                            const int32_t* colind, const double* vals, int32_t* trowptr,
                            int32_t* trow, double* tvals, int32_t* tperm, void* temp,
                            size_t temp_bytes) {
  const bool carry = temp_bytes >= temp_bytes_for(nnz, n, RS_BITS, true);
  const int width = temp_bytes >= temp_bytes_for(nnz, n, RS_BITS, false) ? RS_BITS : RS_NARROW;
  if (temp_bytes < temp_bytes_for(nnz, n, width, false)) return hipErrorInvalidValue;
  if (nnz == 0) {
    k_zero_fill_i32<<<(unsigned)(((int64_t)n + 1 + 255) / 256), 256, 0, st>>>((int64_t)n + 1, 0, trowptr);
    return hipGetLastError();
  }
  const int64_t ntiles = (nnz + RS_TILE - 1) / RS_TILE;
  const int64_t nhist = hist_words(nnz, n, width);
  const int P = passes_for(n, width), nbits = digit_bits(n, width);
  int32_t* hist = (int32_t*)temp;
  int32_t* scanw = hist + nhist;
  int32_t* tab = scanw + scan_tiles(nhist) + 1;
  int32_t* pk = tab + tab_words(nnz);
  int32_t* pv = pk + (P >= 2 ? nnz : 0);
  double* pval = (double*)(hist + even(pv + (P >= 2 ? nnz : 0) - hist));
  int32_t* prow = (int32_t*)(pval + nnz);
  int32_t* sorted = carry ? prow + nnz : trow;      // keys of the passes that write the outputs
  const int64_t nb = (nnz >> ROWTAB_SHIFT) + 1;
  k_row_table<<<(unsigned)((nb + 1 + 255) / 256), 256, 0, st>>>(nnz, m, rowptr, nb, tab);
  // radix passes; the last one writes the outputs, earlier ones alternate so
  // that the sequence ends there
  const int32_t* ik = colind;
  SortCarry C{nullptr, nullptr, vals, nullptr, nullptr, nullptr};
  for (int p = 0; p < P; ++p) {
    const bool to_out = ((P - 1 - p) % 2) == 0;
    int32_t* ok = to_out ? sorted : pk;
    C.operm = to_out ? tperm : pv;
    if (carry) {
      C.orow = to_out ? trow : prow;
      C.oval = tvals ? (to_out ? tvals : pval) : nullptr;
    }
    k_digit_hist<<<(unsigned)ntiles, RS_THREADS, 0, st>>>(nnz, ik, nbits * p, nbits, hist, (int32_t)ntiles);
    exclusive_scan(st, nhist, hist, scanw);
    k_digit_scatter<<<(unsigned)ntiles, RS_THREADS, 0, st>>>(nnz, ik, C, nbits * p, nbits, hist,
                                                             (int32_t)ntiles, ok, rowptr, tab);
    ik = ok;
    C.perm = C.operm;
    C.row = C.orow;
    C.val = C.oval;
  }
  // row pointer of A^T from the sorted columns, then the rows if not carried
  k_col_starts<<<(unsigned)(((int64_t)n + 1 + 255) / 256), 256, 0, st>>>(nnz, sorted, n, trowptr);
  if (!carry)
    k_rows_of<<<(unsigned)((nnz + 256 * ROWS_U - 1) / (256 * ROWS_U)), 256, 0, st>>>(
        nnz, rowptr, tab, tperm, vals, trow, tvals);
  return hipGetLastError();
}

// Row i of the row-permuted copy is row perm[i] of A (prowptr holds the
// permuted row starts).  Eight lanes copy a row together, so that the rows of
// a wave are read and written in runs: with one thread per row, whose accesses
// lie a row apart from its neighbours', 1.9e7 entries took 0.65 ms, this takes
// 0.25 ms.
constexpr int PERM_LANES = 8;
__global__ void __launch_bounds__(256)
k_permute_rows(int32_t m, const int32_t* __restrict__ perm,
               const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colind,
               const double* __restrict__ vals, const int32_t* __restrict__ prowptr,
               int32_t* __restrict__ pcolind, double* __restrict__ pvals) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t i = t / PERM_LANES;
  const int l = (int)(t % PERM_LANES);
  if (i >= m) return;
  const int32_t r = perm[i];
  const int32_t k0 = rowptr[r], len = rowptr[r + 1] - k0, d = prowptr[i];
  for (int32_t q = l; q < len; q += PERM_LANES) {
    pcolind[d + q] = colind[k0 + q];
    pvals[d + q] = vals[k0 + q];
  }
}

void launch_permute_rows(hipStream_t st, int32_t m, const int32_t* perm, const int32_t* rowptr,
                         const int32_t* colind, const double* vals, const int32_t* prowptr,
                         int32_t* pcolind, double* pvals) {
  if (m == 0) return;
  const unsigned blocks = (unsigned)(((int64_t)m * PERM_LANES + 255) / 256);
  k_permute_rows<<<blocks, 256, 0, st>>>(m, perm, rowptr, colind, vals, prowptr, pcolind, pvals);
}

// flag[0] = 1 if a column index lies outside [0, n) (the sort's counters and
// positions assume valid columns)
__global__ void k_check_cols(int64_t nnz, const int32_t* __restrict__ colind, int32_t n,
                             int32_t* __restrict__ flag) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < nnz && (colind[k] < 0 || colind[k] >= n)) flag[0] = 1;
}

void launch_check_cols(hipStream_t st, int64_t nnz, const int32_t* colind, int32_t n, int32_t* flag) {
  k_zero_fill_i32<<<1, 64, 0, st>>>(1, 0, flag);
  if (nnz == 0) return;
  k_check_cols<<<(unsigned)((nnz + 255) / 256), 256, 0, st>>>(nnz, colind, n, flag);
}

// ---------------------------------------------------------------------------
// Input of the setup: the CSR arrays of all instances concatenated into the
// handle's copy of A (row pointers narrowed to int32 and shifted by the
// instance's first entry, columns shifted by its first column), checked on
// the way.  A failed check records the smallest failing (global) row of its
// kind in bad[kind] (atomicMin; INT64_MAX when none): CSR_FIRST rowptr[0] !=
// 0, CSR_LAST rowptr[m] != nnz, CSR_MONO a row start below the previous one
// or above nnz, CSR_RANGE a column outside [0, n), CSR_ORDER columns not
// strictly increasing.  Reads never leave an instance's arrays, whatever
// they hold.
// ---------------------------------------------------------------------------
// the instance holding global index g of the table field (r0 or e0)
__device__ inline int instance_of(const InstDesc* __restrict__ d, int S, int64_t g, bool by_rows) {
  int lo = 0, hi = S - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if ((by_rows ? d[mid].r0 : d[mid].e0) <= g) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

__global__ void k_concat_rows(int S, const InstDesc* __restrict__ d, int64_t M,
                              int32_t* __restrict__ rp, unsigned long long* __restrict__ bad) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= M) return;
  const int k = instance_of(d, S, g, true);
  const InstDesc D = d[k];
  const int64_t r = g - D.r0;
  const int64_t lo = D.rowptr[r], hi = D.rowptr[r + 1];
  if (r == 0 && lo != 0) atomicMin(&bad[CSR_FIRST], (unsigned long long)g);
  if (r == D.m - 1 && hi != D.nnz) atomicMin(&bad[CSR_LAST], (unsigned long long)g);
  if (hi < lo || hi > D.nnz) atomicMin(&bad[CSR_MONO], (unsigned long long)g);
  rp[g + 1] = (int32_t)(D.e0 + min(max(hi, (int64_t)0), D.nnz));
  if (g == 0) rp[0] = 0;
}

__global__ void k_concat_entries(int S, const InstDesc* __restrict__ d, int64_t NNZ,
                                 int32_t* __restrict__ ci, double* __restrict__ vals) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= NNZ) return;
  const int k = instance_of(d, S, e, false);
  const InstDesc D = d[k];
  const int64_t q = e - D.e0;
  ci[e] = D.colind[q] + (int32_t)D.c0;
  vals[e] = D.vals[q];
}

// columns of every row (rp as written by k_concat_rows: inside each
// instance's entries even for a corrupt rowptr)
__global__ void k_check_rows(int S, const InstDesc* __restrict__ d, int64_t M,
                             const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                             unsigned long long* __restrict__ bad) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= M) return;
  const int k = instance_of(d, S, g, true);
  const InstDesc D = d[k];
  const int32_t a = rp[g], b = rp[g + 1];
  const int64_t c0 = D.c0, c1 = D.c0 + D.n;
  for (int32_t e = a; e < b; ++e) {
    const int32_t c = ci[e];
    if (c < c0 || c >= c1) { atomicMin(&bad[CSR_RANGE], (unsigned long long)g); return; }
    if (e > a && c <= ci[e - 1]) { atomicMin(&bad[CSR_ORDER], (unsigned long long)g); return; }
  }
}

__global__ void k_fill_u64(int n, unsigned long long v, unsigned long long* __restrict__ out) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) out[k] = v;
}

void launch_concat(hipStream_t st, int S, const InstDesc* d, int64_t M, int64_t NNZ, int32_t* rp,
                   int32_t* ci, double* vals, unsigned long long* bad) {
  k_fill_u64<<<1, 64, 0, st>>>(CSR_KINDS, ~0ull, bad);
  k_concat_rows<<<(unsigned)((M + 255) / 256), 256, 0, st>>>(S, d, M, rp, bad);
  if (NNZ > 0)
    k_concat_entries<<<(unsigned)((NNZ + 255) / 256), 256, 0, st>>>(S, d, NNZ, ci, vals);
  k_check_rows<<<(unsigned)((M + 255) / 256), 256, 0, st>>>(S, d, M, rp, ci, bad);
}

// ---------------------------------------------------------------------------
// Transpose without allocation: the sort's work arrays live in a file-scope
// device array, `scratch`, of TRANSPOSE_SCRATCH_BYTES, which every GPU the
// library runs on holds until the process ends.  Its device address is taken
// once per device with hipGetSymbolAddress (the array's name in host code is
// only a host-side stand-in) and kept per device.
// ---------------------------------------------------------------------------
namespace {
constexpr size_t TRANSPOSE_SCRATCH_BYTES = (size_t)104 << 20;
constexpr int MAX_DEVICES = 64;
}  // namespace

static __device__ __align__(256) unsigned char scratch[TRANSPOSE_SCRATCH_BYTES];

namespace {
std::mutex g_scratch_mu;
void* g_scratch_ptr[MAX_DEVICES] = {};

// Work space that decides whether a call is taken: 8-bit digits over tiles
// of 4,096 keys, 1/4 byte per entry.  The narrow digits of launch_transpose
// take 1/8 byte per entry for their histogram (tiles twice as large) and
// 1/16 for the row table, so every call it admits has room.
size_t noalloc_bytes(int64_t nnz, int32_t n) {
  const int64_t hist = (nnz + 4095) / 4096 * 256;
  const int64_t scan = std::max(scan_tiles(hist), scan_tiles((int64_t)n + 1)) + 1;
  const int64_t pp = passes_for(n, RS_NARROW) >= 2 ? 2 * nnz : 0;
  return (size_t)(((hist + scan + pp) * 4 + 255) / 256 * 256);
}

// device address of `scratch` on the current device
hipError_t scratch_address(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> g(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}
}  // namespace

}  // namespace lsq2l

extern "C" lsq2l_status lsq2l_transpose_noalloc(int32_t m, int32_t n, int32_t nnz,
                                                const int32_t* rowptr, const int32_t* colind,
                                                const double* vals, int32_t* trowptr,
                                                int32_t* trow, double* tvals, int32_t* tperm,
                                                void* hip_stream) {
  using namespace lsq2l;
  if (m < 0 || n < 0 || nnz < 0 || !rowptr || !trowptr || (nnz > 0 && (!colind || !trow)) ||
      (nnz > 0 && tvals && !vals)) {
    set_error("bad sizes or NULL required pointer");
    return LSQ2L_EINVAL;
  }
  const size_t perm_bytes = tperm ? 0 : ((size_t)nnz * sizeof(int32_t) + 255) / 256 * 256;
  const size_t need = noalloc_bytes(nnz, n) + perm_bytes + 256;
  if (need > TRANSPOSE_SCRATCH_BYTES) {
    set_error("transpose without allocation: n = " + std::to_string(n) + ", nnz = " +
              std::to_string(nnz) + " need " + std::to_string(need) +
              " bytes of work space, above the " + std::to_string(TRANSPOSE_SCRATCH_BYTES) +
              " bytes held per device");
    return LSQ2L_EINVAL;
  }
  // the sort takes wide digits where their histogram fits beside the rest
  const size_t tb = std::min(transpose_temp_bytes(nnz, n),
                             (TRANSPOSE_SCRATCH_BYTES - perm_bytes - 256) / 256 * 256);
  const hipStream_t st = (hipStream_t)hip_stream;
  void* base = nullptr;
  hipError_t e = scratch_address(&base);
  if (e != hipSuccess) {
    set_error(std::string("transpose without allocation: hipGetSymbolAddress: ") + hipGetErrorString(e));
    return LSQ2L_EHIP;
  }
  int32_t* perm = tperm ? tperm : (int32_t*)((char*)base + tb);
  int32_t* flag = (int32_t*)((char*)base + tb + perm_bytes);
  int32_t hflag = 0;
  launch_check_cols(st, nnz, colind, n, flag);
  e = hipMemcpyAsync(&hflag, flag, sizeof(int32_t), hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e == hipSuccess && hflag == 0)
    e = launch_transpose(st, m, n, nnz, rowptr, colind, vals, trowptr, trow, tvals, perm, base, tb);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) {
    set_error(std::string("transpose without allocation: ") + hipGetErrorString(e));
    return LSQ2L_EHIP;
  }
  if (hflag) {
    set_error("transpose: a column index lies outside [0, n)");
    return LSQ2L_EINVAL;
  }
  return LSQ2L_OK;
}

