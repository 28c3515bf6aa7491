// Kernels of the device planner (plan_dev.cpp): the index sets, envelopes and
// overlap maps that plan_build and plan_maps form on the host, found by
// stable sorts of (row, part) and (column, part) pairs (launch_transpose) with
// the passes below between them.
//
// What bounds it: the bytes of the sorts and the gathers of the entries' parts.
// Planning phase, with the transpose of A: 2.7e7 entries in 9e6 rows (64
// banded instances) 5.4 ms, of which sorts 2.6 (16 ms on sixteen host threads);
// 1.9e7 entries, irregular, 3.4 (25); a grid of 1e6 columns 1.7 (8.8).
#include "kernels.hpp"

namespace lsq2l {

constexpr int RL = 4, CL = 8;                      // lanes of a row, of a column
constexpr int SEG_MAX_Y = 1024;

__global__ void k_iota(int64_t n, int32_t* __restrict__ out) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) out[k] = (int32_t)k;
}

// position of every column in its part (pcols: columns by part, ascending)
__global__ void k_locown(int32_t n, const int32_t* __restrict__ pcols, const int32_t* __restrict__ part,
                         const int32_t* __restrict__ pptr, int32_t* __restrict__ locown) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int32_t c = pcols[k];
  locown[c] = (int32_t)k - pptr[part[c]];
}

// The runs of equal parts along the entries of every row: their number
// (ptr[r], and 0 at r = m), or with FILL their parts at out[ptr[r] ..].
template <bool FILL>
__global__ void k_row_runs(int32_t m, const int32_t* __restrict__ rowptr, const int2* __restrict__ owner,
                           int32_t* __restrict__ ptr, int32_t* __restrict__ out) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t r = t / RL;
  const int l = (int)(t % RL);
  if (r > m) return;
  int run = 0;
  if (r < m) {
    const int32_t a = rowptr[r], b = rowptr[r + 1];
    const int32_t at = FILL ? ptr[r] : 0;
    for (int32_t e0 = a; e0 < b; e0 += RL) {
      const int32_t e = e0 + l;
      const int32_t w = e < b ? owner[e].x : -1;
      const bool f = e < b && (e == a || owner[e - 1].x != w);
      const uint32_t g = (uint32_t)(__ballot(f) >> (threadIdx.x % 64 & ~(RL - 1))) & ((1u << RL) - 1u);
      if (FILL && f) out[at + run + __popc(g & ((1u << l) - 1u))] = w;
      run += __popc(g);
    }
  }
  if (!FILL && l == 0) ptr[r] = run;
}

// first[k] = 1 where key[k] (ascending inside segment i = [ptr[i], ptr[i+1]))
// differs from the key before it in its segment; first[ptr[nseg]] = 0
__global__ void k_seg_first(int32_t nseg, const int32_t* __restrict__ ptr, const int32_t* __restrict__ key,
                            int32_t* __restrict__ first) {
  const int32_t i = blockIdx.x, a = ptr[i], b = ptr[i + 1];
  for (int64_t k = a + (int64_t)blockIdx.y * blockDim.x + threadIdx.x; k < b; k += (int64_t)blockDim.x * gridDim.y)
    first[k] = k == a || key[k] != key[k - 1];
  if (i == nseg - 1 && blockIdx.y == 0 && threadIdx.x == 0) first[b] = 0;
}

// the distinct keys of every segment, at = exclusive scan of first, and the
// segments' new extents
__global__ void k_seg_pack(int32_t nseg, const int32_t* __restrict__ ptr, const int32_t* __restrict__ key,
                           const int32_t* __restrict__ at, int32_t* __restrict__ out,
                           int32_t* __restrict__ optr) {
  const int32_t i = blockIdx.x, a = ptr[i], b = ptr[i + 1];
  for (int64_t k = a + (int64_t)blockIdx.y * blockDim.x + threadIdx.x; k < b; k += (int64_t)blockDim.x * gridDim.y)
    if (at[k + 1] != at[k]) out[at[k]] = key[k];
  if (blockIdx.y == 0 && threadIdx.x == 0) {
    optr[i] = at[a];
    if (i == nseg - 1) optr[nseg] = at[b];
  }
}

// sum of the block's threads' v (a maximum with MAX), valid in thread 0
template <bool MAX>
__device__ inline unsigned long long block_fold(unsigned long long v, unsigned long long* sh) {
  auto fold = [](unsigned long long x, unsigned long long y) { return MAX ? (x > y ? x : y) : x + y; };
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fold(v, __shfl_xor(v, o, 64));
  if (threadIdx.x % 64 == 0) sh[threadIdx.x / 64] = v;
  __syncthreads();
  for (int w = 1; w < 4; ++w) v = fold(v, sh[w]);
  __syncthreads();
  return v;
}

// stat[0] = longest row and column of A; stat[1] += rows whose first column
// (n: empty row) lies more than jump below that of the row before
__global__ void __launch_bounds__(256)
k_plan_stat(int32_t m, int32_t n, const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colind,
            const int32_t* __restrict__ trowptr, int32_t jump, unsigned long long* __restrict__ stat) {
  __shared__ unsigned long long sh[4];
  unsigned long long L = 0, c = 0;
  const int64_t step = (int64_t)blockDim.x * gridDim.x, t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (int64_t r = t0; r < m; r += step) {
    const int32_t a = rowptr[r], b = rowptr[r + 1], p = r > 0 ? rowptr[r - 1] : a;
    L = max(L, (unsigned long long)(b - a));
    if (r > 0 && (a < b ? colind[a] : n) < (p < a ? colind[p] : n) - jump) ++c;
  }
  for (int64_t k = t0; k < n; k += step) L = max(L, (unsigned long long)(trowptr[k + 1] - trowptr[k]));
  L = block_fold<true>(L, sh);
  c = block_fold<false>(c, sh);
  if (threadIdx.x == 0) {
    atomicMax(&stat[0], L);
    if (c) atomicAdd(&stat[1], c);
  }
}

// With k > 1 parts in a row of L entries: size[0] += L (k - 1), size[1] +=
// k (k - 1) / 2 over the rows, size[2] = largest L k
__global__ void __launch_bounds__(256)
k_plan_size(int32_t m, const int32_t* __restrict__ rowptr, const int32_t* __restrict__ qptr,
            unsigned long long* __restrict__ size) {
  __shared__ unsigned long long sh[4];
  unsigned long long c = 0, p = 0, w = 0;
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < m; r += (int64_t)blockDim.x * gridDim.x) {
    const unsigned long long L = rowptr[r + 1] - rowptr[r];
    const unsigned long long k = qptr[r + 1] - qptr[r];
    if (k < 2) continue;
    c += L * (k - 1);
    p += k * (k - 1) / 2;
    w = max(w, L * k);
  }
  c = block_fold<false>(c, sh);
  p = block_fold<false>(p, sh);
  w = block_fold<true>(w, sh);
  if (threadIdx.x == 0 && c) {
    atomicAdd(&size[0], c);
    atomicAdd(&size[1], p);
    atomicMax(&size[2], w);
  }
}

// The parts other than a column's own met along the rows of every column
// (repeats included): their number (ptr[c], and 0 at c = n), or with FILL
// the parts at out[ptr[c] ..].
template <bool FILL>
__global__ void k_col_parts(int32_t n, const int32_t* __restrict__ trowptr, const int32_t* __restrict__ trow,
                            const int32_t* __restrict__ qptr, const int32_t* __restrict__ qpart,
                            const int32_t* __restrict__ part, int32_t* __restrict__ ptr,
                            int32_t* __restrict__ out) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t c = t / CL;
  const int l = (int)(t % CL);
  if (c > n) return;
  int run = 0;
  if (c < n) {
    const int32_t a = trowptr[c], b = trowptr[c + 1];
    const int32_t at = FILL ? ptr[c] : 0, own = FILL ? part[c] : 0;
    for (int32_t k0 = a; k0 < b; k0 += CL) {
      int32_t q0 = 0, k = 0;
      if (k0 + l < b) {
        const int32_t r = trow[k0 + l];
        q0 = qptr[r];
        k = qptr[r + 1] - q0 - 1;                  // the column's own part is one of them
      }
      int x = k;
#pragma unroll
      for (int o = 1; o < CL; o <<= 1) {
        const int y = __shfl_up(x, o, CL);
        if (l >= o) x += y;
      }
      if (FILL) {
        int w = at + run + x - k;
        for (int q = 0; q <= k && k > 0; ++q)
          if (qpart[q0 + q] != own) out[w++] = qpart[q0 + q];
      }
      run += __shfl(x, CL - 1, CL);
    }
  }
  if (!FILL && l == 0) ptr[c] = run;
}

// Omega_i = Omega_Ii, Omega_Gamma_i; tile envelope started at the diagonal
__global__ void k_plan_omega(const SubDesc* __restrict__ subs, const int32_t* __restrict__ pptr,
                             const int32_t* __restrict__ pcols, const int32_t* __restrict__ goff,
                             const int32_t* __restrict__ gamma, int32_t* __restrict__ omega,
                             int32_t* __restrict__ F) {
  const int i = blockIdx.x;
  const SubDesc d = subs[i];
  const int step = blockDim.x * gridDim.y, t0 = blockIdx.y * blockDim.x + threadIdx.x;
  for (int a = t0; a < d.nI; a += step) omega[d.omega_off + a] = pcols[pptr[i] + a];
  for (int a = t0; a < d.nG; a += step) omega[d.omega_off + d.nI + a] = gamma[goff[i] + a];
  for (int a = t0; a < d.ntiles; a += step) F[d.tile_base + a] = a;
}

// Tile envelope of every C_ii: a row of Xi_i couples all its positions, so its
// least position bounds the tile rows of all of them.  RL lanes walk a row,
// once per part it holds; a bound that already holds is read only.
__global__ void k_plan_envelope(int32_t m, const int32_t* __restrict__ qptr, const int32_t* __restrict__ qpart,
                                const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colind,
                                const int2* __restrict__ owner, const SubDesc* __restrict__ subs,
                                const int32_t* __restrict__ goff, const int32_t* __restrict__ gamma,
                                int32_t* __restrict__ F) {
  const int64_t r = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / RL;
  const int l = threadIdx.x % RL;
  if (r >= m) return;
  const int32_t a = rowptr[r], b = rowptr[r + 1];
  const int2 mine = a + l < b ? owner[a + l] : int2{-1, 0};
  for (int32_t q = qptr[r]; q < qptr[r + 1]; ++q) {
    const int i = qpart[q];
    const int32_t nIp = subs[i].nIp, g0 = goff[i], nG = goff[i + 1] - g0;
    const int64_t tb = subs[i].tile_base;
    auto position = [&](int32_t e, int2 w) -> int32_t {
      if (w.x == i) return w.y;
      const int32_t c = colind[e];
      int32_t lo = 0, hi = nG;
      while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if (gamma[g0 + mid] < c) lo = mid + 1; else hi = mid;
      }
      return nIp + lo;                             // every column of a row of Xi_i is in Omega_i
    };
    int32_t best = INT32_MAX, first = 0;
    if (a + l < b) best = first = position(a + l, mine);
    for (int32_t e = a + l + RL; e < b; e += RL) best = min(best, position(e, owner[e]));
#pragma unroll
    for (int o = RL / 2; o > 0; o >>= 1) best = min(best, __shfl_xor(best, o, RL));
    best /= TS;
    for (int32_t e = a + l; e < b; e += RL) {
      const int32_t p = e == a + l ? first : position(e, owner[e]);
      if (F[tb + p / TS] > best) atomicMin(&F[tb + p / TS], best);
    }
  }
}

// offsets of the stored tile rows of every subdomain and its stored tiles; a
// wave per subdomain
__global__ void __launch_bounds__(64)
k_tile_offsets(const SubDesc* __restrict__ subs, const int32_t* __restrict__ F, int64_t* __restrict__ off,
               int64_t* __restrict__ stored) {
  const SubDesc d = subs[blockIdx.x];
  const int lane = threadIdx.x;
  int64_t run = 0;
  for (int32_t t0 = 0; t0 < d.ntiles; t0 += 64) {
    const int32_t t = t0 + lane;
    const int64_t v = t < d.ntiles ? t - F[d.tile_base + t] + 1 : 0;
    int64_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int64_t y = __shfl_up(x, o, 64);
      if (lane >= o) x += y;
    }
    if (t < d.ntiles) off[d.tile_base + t] = run + x - v;
    run += __shfl(x, 63, 64);
  }
  if (lane == 0) stored[blockIdx.x] = run;
}

// Inverse overlap map: the local positions holding column c, by increasing
// subdomain: its own part's, and those of the interfaces that hold it
// (optr, opart, operm: the lists Omega_Gamma_i sorted by column).
__global__ void k_own_maps(int32_t n, const int32_t* __restrict__ part, const int32_t* __restrict__ locown,
                           const SubDesc* __restrict__ subs, const int32_t* __restrict__ goff,
                           const int32_t* __restrict__ optr, const int32_t* __restrict__ opart,
                           const int32_t* __restrict__ operm, int32_t* __restrict__ own_ptr,
                           int32_t* __restrict__ own_pos) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c > n) return;
  const int32_t o0 = optr[c];
  own_ptr[c] = (int32_t)(o0 + c);
  if (c == n) return;
  const int32_t o1 = optr[c + 1], w = part[c];
  int64_t at = o0 + c;
  bool done = false;
  for (int32_t o = o0; o < o1; ++o) {
    const int32_t j = opart[o];
    if (!done && j > w) {
      own_pos[at++] = (int32_t)subs[w].loc_off + locown[c];
      done = true;
    }
    own_pos[at++] = (int32_t)subs[j].loc_off + subs[j].nIp + operm[o] - goff[j];
  }
  if (!done) own_pos[at] = (int32_t)subs[w].loc_off + locown[c];
}

// Pairs of parts sharing a row, in row order, as (i, j, place of the row in
// Xi_i, in Xi_j): entry t of the list of (row, part) pairs meets the later
// entries of its row
__global__ void k_pair_count(int64_t nx, const int32_t* __restrict__ xi, const int32_t* __restrict__ qperm,
                             const int32_t* __restrict__ qptr, int32_t* __restrict__ cnt) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t > nx) return;
  cnt[t] = t < nx ? qptr[xi[qperm[t]] + 1] - (int32_t)t - 1 : 0;
}
__global__ void k_pair_fill(int64_t nx, const int32_t* __restrict__ qperm, const int32_t* __restrict__ qpart,
                            const int32_t* __restrict__ xoff, const int32_t* __restrict__ at,
                            int4* __restrict__ rec) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= nx) return;
  const int32_t a = at[t], k = at[t + 1] - a;
  if (k == 0) return;
  const int32_t i = qpart[t], ri = qperm[t] - xoff[i];
  for (int32_t v = 0; v < k; ++v) {
    const int32_t j = qpart[t + 1 + v];
    rec[a + v] = int4{i, j, ri, qperm[t + 1 + v] - xoff[j]};
  }
}

// first column of every row (n: empty row)
__global__ void k_row_keys(int32_t m, int32_t n, const int32_t* __restrict__ rowptr,
                           const int32_t* __restrict__ colind, int32_t* __restrict__ key) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r < m) key[r] = rowptr[r] < rowptr[r + 1] ? colind[rowptr[r]] : n;
}

// lengths of the rows in the order perm, 0 at m
__global__ void k_perm_len(int32_t m, const int32_t* __restrict__ perm, const int32_t* __restrict__ rowptr,
                           int32_t* __restrict__ len) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k > m) return;
  len[k] = k < m ? rowptr[perm[k] + 1] - rowptr[perm[k]] : 0;
}

// ---------------------------------------------------------------------------
static unsigned blocks_of(int64_t threads) { return (unsigned)((threads + 255) / 256); }
static dim3 seg_grid(int32_t nseg, int64_t len) {
  const int64_t per = len / ((int64_t)nseg * 1024) + 1;
  return dim3((unsigned)nseg, (unsigned)(per < SEG_MAX_Y ? per : SEG_MAX_Y));
}

void launch_iota(hipStream_t st, int64_t n, int32_t* out) {
  k_iota<<<blocks_of(n), 256, 0, st>>>(n, out);
}
void launch_locown(hipStream_t st, int32_t n, const int32_t* pcols, const int32_t* part, const int32_t* pptr,
                   int32_t* locown) {
  k_locown<<<blocks_of(n), 256, 0, st>>>(n, pcols, part, pptr, locown);
}
void launch_row_runs(hipStream_t st, int32_t m, const int32_t* rowptr, const int2* owner, int32_t* ptr,
                     int32_t* out) {
  const unsigned nb = blocks_of(((int64_t)m + 1) * RL);
  if (out) k_row_runs<true><<<nb, 256, 0, st>>>(m, rowptr, owner, ptr, out);
  else k_row_runs<false><<<nb, 256, 0, st>>>(m, rowptr, owner, ptr, out);
}
void launch_seg_first(hipStream_t st, int32_t nseg, int64_t len, const int32_t* ptr, const int32_t* key,
                      int32_t* first) {
  k_seg_first<<<seg_grid(nseg, len), 256, 0, st>>>(nseg, ptr, key, first);
}
void launch_seg_pack(hipStream_t st, int32_t nseg, int64_t len, const int32_t* ptr, const int32_t* key,
                     const int32_t* at, int32_t* out, int32_t* optr) {
  k_seg_pack<<<seg_grid(nseg, len), 256, 0, st>>>(nseg, ptr, key, at, out, optr);
}
void launch_plan_stat(hipStream_t st, const DevMatrix& M, int32_t jump, unsigned long long* stat) {
  const unsigned nb = blocks_of(M.m);
  k_plan_stat<<<nb < 1024 ? nb : 1024, 256, 0, st>>>(M.m, M.n, M.rowptr, M.colind, M.trowptr, jump, stat);
}
void launch_plan_size(hipStream_t st, int32_t m, const int32_t* rowptr, const int32_t* qptr,
                      unsigned long long* size) {
  const unsigned nb = blocks_of(m);
  k_plan_size<<<nb < 1024 ? nb : 1024, 256, 0, st>>>(m, rowptr, qptr, size);
}
void launch_col_parts(hipStream_t st, int32_t n, const int32_t* trowptr, const int32_t* trow,
                      const int32_t* qptr, const int32_t* qpart, const int32_t* part, int32_t* ptr,
                      int32_t* out) {
  const unsigned nb = blocks_of(((int64_t)n + 1) * CL);
  if (out) k_col_parts<true><<<nb, 256, 0, st>>>(n, trowptr, trow, qptr, qpart, part, ptr, out);
  else k_col_parts<false><<<nb, 256, 0, st>>>(n, trowptr, trow, qptr, qpart, part, ptr, out);
}
void launch_plan_omega(hipStream_t st, int32_t nsub, const SubDesc* subs, const int32_t* pptr,
                       const int32_t* pcols, const int32_t* goff, const int32_t* gamma, int32_t* omega,
                       int32_t* F) {
  k_plan_omega<<<dim3((unsigned)nsub, 4), 256, 0, st>>>(subs, pptr, pcols, goff, gamma, omega, F);
}
void launch_plan_envelope(hipStream_t st, const int32_t* qptr, const int32_t* qpart, const DevMatrix& M,
                          const int2* owner, const SubDesc* subs, const int32_t* goff,
                          const int32_t* gamma, int32_t* F) {
  k_plan_envelope<<<blocks_of((int64_t)M.m * RL), 256, 0, st>>>(M.m, qptr, qpart, M.rowptr, M.colind, owner,
                                                                subs, goff, gamma, F);
}
void launch_tile_offsets(hipStream_t st, int32_t nsub, const SubDesc* subs, const int32_t* F, int64_t* off,
                         int64_t* stored) {
  k_tile_offsets<<<(unsigned)nsub, 64, 0, st>>>(subs, F, off, stored);
}
void launch_own_maps(hipStream_t st, int32_t n, const int32_t* part, const int32_t* locown,
                     const SubDesc* subs, const int32_t* goff, const int32_t* optr, const int32_t* opart,
                     const int32_t* operm, int32_t* own_ptr, int32_t* own_pos) {
  k_own_maps<<<blocks_of((int64_t)n + 1), 256, 0, st>>>(n, part, locown, subs, goff, optr, opart, operm,
                                                        own_ptr, own_pos);
}
void launch_pair_count(hipStream_t st, int64_t nx, const int32_t* xi, const int32_t* qperm,
                       const int32_t* qptr, int32_t* cnt) {
  k_pair_count<<<blocks_of(nx + 1), 256, 0, st>>>(nx, xi, qperm, qptr, cnt);
}
void launch_pair_fill(hipStream_t st, int64_t nx, const int32_t* qperm, const int32_t* qpart,
                      const int32_t* xoff, const int32_t* at, int4* rec) {
  if (nx == 0) return;
  k_pair_fill<<<blocks_of(nx), 256, 0, st>>>(nx, qperm, qpart, xoff, at, rec);
}
void launch_row_keys(hipStream_t st, int32_t m, int32_t n, const int32_t* rowptr, const int32_t* colind,
                     int32_t* key) {
  k_row_keys<<<blocks_of(m), 256, 0, st>>>(m, n, rowptr, colind, key);
}
void launch_perm_len(hipStream_t st, int32_t m, const int32_t* perm, const int32_t* rowptr, int32_t* len) {
  k_perm_len<<<blocks_of((int64_t)m + 1), 256, 0, st>>>(m, perm, rowptr, len);
}

}  // namespace lsq2l
