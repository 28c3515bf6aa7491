// Sparse products and the vector work of preconditioned CG on C = A^T A
// (eq. normal): C p is applied as A^T (A p), never formed.
//
// Reductions are deterministic: every segment (instance) of a vector is cut
// into chunks by its length and that of the whole vector alone, each reduced by a
// fixed tree; the workgroup that finishes a segment last adds the chunks' sums
// by another fixed tree and takes the step that needs the sum.  Repeated runs
// give bitwise-identical results.
#include <algorithm>
#include <type_traits>

#include "kernels.hpp"

namespace lsq2l {

// y = A x, G lanes per row (G in {1, 2, 4, 8, 16, 32, 64}); rows are short
// (1 - 64 stored entries), so a sub-wave per row keeps lanes busy and the
// column/value reads coalesced inside the group.
template <int G>
__global__ void __launch_bounds__(256)
k_spmv(int32_t nrows, const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colind,
       const double* __restrict__ vals, const double* __restrict__ x, double* __restrict__ y) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t row = t / G;
  const int sub = (int)(t % G);
  double s = 0.0;
  if (row < nrows) {
    const int e1 = rowptr[row + 1];
    for (int e = rowptr[row] + sub; e < e1; e += G) s += vals[e] * x[colind[e]];
  }
#pragma unroll
  for (int w = G / 2; w > 0; w /= 2) s += __shfl_down(s, w, G);
  if (row < nrows && sub == 0) y[row] = s;
}

// y = A x for short, uneven rows, staged through LDS.  Workgroup b owns the
// rows whose first entry lies in [b SPMV_NB, (b + 1) SPMV_NB): rows
// tab[2b] .. tab[2b + 2] - 1, whose entries start at tab[2b + 1] (a table
// made once per matrix, k_row_blocks), so that one 8-byte load gives the
// block's extent.  Its entries are read once, coalesced, four per thread in
// flight, as vals[e] x[colind[e]] into LDS; then every thread sums its rows
// from LDS in entry order and writes y coalesced.  A block whose rows hold
// more than SPMV_CAP entries (a long last row) sums each row with a
// wavefront instead.  Every row is summed in one fixed order, so runs are
// bitwise reproducible.  With STREAM the matrix arrays are read with
// non-temporal loads, which keeps the caches for x when the matrix is
// larger than the last-level cache.
constexpr int SPMV_NB = 1024, SPMV_CAP = 2048, SPMV_THREADS = 256, SPMV_U = 4;
constexpr int64_t SPMV_STREAM_BYTES = (int64_t)256 << 20;   // MI355X last-level cache

int64_t spmv_blocks(int64_t nnz) { return std::max<int64_t>(1, (nnz + SPMV_NB - 1) / SPMV_NB); }
int64_t spmv_table_len(int64_t nnz) { return 2 * (spmv_blocks(nnz) + 1); }

// tab[2b] = first row whose start is >= b SPMV_NB (b < nblk), tab[2b + 1] =
// its start; tab[2 nblk] = nrows, tab[2 nblk + 1] = nnz
__global__ void k_row_blocks(int32_t nrows, const int32_t* __restrict__ rowptr, int64_t nblk,
                             int32_t* __restrict__ tab) {
  const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (b > nblk) return;
  int32_t lo = nrows;
  if (b < nblk) {
    const int64_t v = b * SPMV_NB;
    lo = 0;
    int32_t hi = nrows;
    while (lo < hi) {
      const int32_t mid = (int32_t)(((int64_t)lo + hi) >> 1);
      if (rowptr[mid] < v) lo = mid + 1;
      else hi = mid;
    }
  }
  tab[2 * b] = lo;
  tab[2 * b + 1] = rowptr[lo];
}

void launch_row_blocks(hipStream_t st, int32_t nrows, const int32_t* rowptr, int64_t nnz, int32_t* tab) {
  const int64_t nblk = spmv_blocks(nnz);
  k_row_blocks<<<(unsigned)((nblk + 1 + 255) / 256), 256, 0, st>>>(nrows, rowptr, nblk, tab);
}

template <bool STREAM, typename V>
__device__ inline V spmv_load(const V* p) {
  if constexpr (STREAM) return __builtin_nontemporal_load(p);
  else return *p;
}

template <bool STREAM, bool PLACED>
__global__ void __launch_bounds__(SPMV_THREADS)
k_spmv_stream(const int32_t* __restrict__ tab, const int32_t* __restrict__ rowptr,
              const int32_t* __restrict__ colind, const double* __restrict__ vals,
              const double* __restrict__ x, double* __restrict__ y, const int32_t* __restrict__ place) {
  __shared__ double prod[SPMV_CAP];
  const int tid = threadIdx.x;
  typedef int32_t i2 __attribute__((ext_vector_type(2)));
  const i2 lo = reinterpret_cast<const i2*>(tab)[blockIdx.x];
  const i2 hi = reinterpret_cast<const i2*>(tab)[blockIdx.x + 1];
  const int32_t r0 = lo.x, e0 = lo.y, r1 = hi.x, e1 = hi.y;
  if (r0 >= r1) return;
  if (e1 - e0 <= SPMV_CAP) {
    for (int32_t e = e0 + tid; e < e1; e += SPMV_U * SPMV_THREADS) {
      int32_t c[SPMV_U];
      double v[SPMV_U];
#pragma unroll
      for (int u = 0; u < SPMV_U; ++u) {
        const int32_t q = e + u * SPMV_THREADS;
        c[u] = q < e1 ? spmv_load<STREAM>(colind + q) : 0;
        v[u] = q < e1 ? spmv_load<STREAM>(vals + q) : 0.0;
      }
#pragma unroll
      for (int u = 0; u < SPMV_U; ++u) {
        const int32_t q = e + u * SPMV_THREADS;
        if (q < e1) prod[q - e0] = v[u] * x[c[u]];
      }
    }
    __syncthreads();
    for (int32_t r = r0 + tid; r < r1; r += SPMV_THREADS) {
      const int32_t a = rowptr[r] - e0, b = rowptr[r + 1] - e0;
      double s = 0.0;
      for (int32_t k = a; k < b; ++k) s += prod[k];
      y[PLACED ? place[r] : r] = s;
    }
    return;
  }
  // long rows: one wavefront per row, lanes strided over the row
  const int lane = tid & 63, wave = tid >> 6;
  for (int32_t r = r0 + wave; r < r1; r += SPMV_THREADS / 64) {
    double s = 0.0;
    for (int32_t e = rowptr[r] + lane; e < rowptr[r + 1]; e += 64) s += vals[e] * x[colind[e]];
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) s += __shfl_down(s, w, 64);
    if (lane == 0) y[PLACED ? place[r] : r] = s;
  }
}

// out[i] = in[perm[i]]; bound by the lines that the scattered reads touch
__global__ void __launch_bounds__(256)
k_gather(int64_t n, const int32_t* __restrict__ perm, const double* __restrict__ in, double* __restrict__ out) {
  const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (k < n) out[k] = in[perm[k]];
}

void launch_gather(hipStream_t st, int64_t n, const int32_t* perm, const double* in, double* out) {
  if (n == 0) return;
  k_gather<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(n, perm, in, out);
}

// with place, row r of the product goes to y[place[r]] (row blocks only)
// group 0: row blocks, streaming loads if the matrix arrays (12 bytes per
// entry) exceed the last-level cache; -1 / -2: row blocks with cached /
// streaming loads; 1 .. 64: that many lanes per row
void launch_spmv(hipStream_t st, int32_t nrows, const int32_t* rowptr, const int32_t* colind,
                 const double* vals, const double* x, double* y, int group, int64_t nnz,
                 const int32_t* blk, const int32_t* place) {
  if (nrows == 0) return;
  if (group == 0) group = 12 * nnz > SPMV_STREAM_BYTES ? SPMV_ROWS_STREAM : SPMV_ROWS_CACHED;
  if (group < 0 && blk) {
    const bool str = group == SPMV_ROWS_STREAM;
    auto* kernel = place ? (str ? k_spmv_stream<true, true> : k_spmv_stream<false, true>)
                         : (str ? k_spmv_stream<true, false> : k_spmv_stream<false, false>);
    kernel<<<(unsigned)spmv_blocks(nnz), SPMV_THREADS, 0, st>>>(blk, rowptr, colind, vals, x, y, place);
    return;
  }
  if (group < 0) group = 1;
  const int64_t threads = (int64_t)nrows * group;
  const unsigned blocks = (unsigned)((threads + 255) / 256);
  switch (group) {
    case 1: k_spmv<1><<<blocks, 256, 0, st>>>(nrows, rowptr, colind, vals, x, y); break;
    case 2: k_spmv<2><<<blocks, 256, 0, st>>>(nrows, rowptr, colind, vals, x, y); break;
    case 4: k_spmv<4><<<blocks, 256, 0, st>>>(nrows, rowptr, colind, vals, x, y); break;
    case 8: k_spmv<8><<<blocks, 256, 0, st>>>(nrows, rowptr, colind, vals, x, y); break;
    case 16: k_spmv<16><<<blocks, 256, 0, st>>>(nrows, rowptr, colind, vals, x, y); break;
    case 32: k_spmv<32><<<blocks, 256, 0, st>>>(nrows, rowptr, colind, vals, x, y); break;
    default: k_spmv<64><<<blocks, 256, 0, st>>>(nrows, rowptr, colind, vals, x, y); break;
  }
}

// dL/dA_ij = r_i lam_j - (A lam)_i x_j on the stored pattern, CSR order.
__global__ void k_grad_vals(int32_t m, const int32_t* __restrict__ rowptr,
                            const int32_t* __restrict__ colind, const double* __restrict__ r,
                            const double* __restrict__ lam, const double* __restrict__ Alam,
                            const double* __restrict__ x, double* __restrict__ out) {
  const int row = blockIdx.x * blockDim.x + threadIdx.x;
  if (row >= m) return;
  const double ri = r[row], ai = Alam[row];
  for (int e = rowptr[row]; e < rowptr[row + 1]; ++e) {
    const int j = colind[e];
    out[e] = ri * lam[j] - ai * x[j];
  }
}

void launch_grad_vals(hipStream_t st, int32_t m, const int32_t* rowptr, const int32_t* colind,
                      const double* r, const double* lam, const double* Alam, const double* x,
                      double* out) {
  if (m == 0) return;
  k_grad_vals<<<(m + 255) / 256, 256, 0, st>>>(m, rowptr, colind, r, lam, Alam, x, out);
}

// Sum over a block of 256 threads: a sum in every wave, then the four wave
// sums in order (the result is returned to every thread)
__device__ inline double block_reduce_256(double v, double* sh) {
  v = wave_allsum(v);
  const int wave = threadIdx.x / 64;
  __syncthreads();
  if (threadIdx.x % 64 == 0) sh[wave] = v;
  __syncthreads();
  return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// The step of the Krylov methods that follows a sum (one thread per segment):
// v is the sum, v2 the second one where the reduction has two.
__device__ inline void reduction_step(const Reduction& R, int s, double v, double v2) {
  const Scalars& sc = R.sc;
  double* ls = R.lsqr + (int64_t)s * LSQR_NSC;
  switch (R.op) {
    case OP_SUM:
      R.out[s] = v;
      break;
    case OP_R0:
      sc.r0n2[s] = v;
      sc.rn2[s] = v;
      sc.its[s] = 0;
      sc.done[s] = (v == 0.0) ? 1 : 0;
      break;
    case OP_RHO_INIT:
      sc.rho[s] = v;
      if (sc.done[s] == 0 && !isfinite(v)) sc.done[s] = 2;
      break;
    case OP_ALPHA:
      sc.pq[s] = v;
      if (sc.done[s] != 0) {
        sc.alpha[s] = 0.0;
      } else if (!(v > 0.0) || !isfinite(v) || !isfinite(sc.rho[s])) {
        sc.alpha[s] = 0.0;
        sc.done[s] = 2;
      } else {
        sc.alpha[s] = sc.rho[s] / v;
        sc.its[s] += 1;
      }
      break;
    case OP_RNORM: {
      sc.rn2[s] = v;
      int dn = sc.done[s];
      if (dn == 0) {
        if (!isfinite(v)) dn = 2;
        else if (v <= R.tol * sc.r0n2[s]) dn = 1;
        sc.done[s] = dn;
      }
      // the host reads the flag after the next synchronization
      __hip_atomic_store(&sc.h_done[s], dn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      break;
    }
    case OP_BETA: {
      // v: z^T r_new; v2 (flexible only): z^T r_old
      const double num = R.two ? (v - v2) : v;
      if (sc.done[s] != 0) sc.beta[s] = 0.0;
      else sc.beta[s] = num / sc.rho[s];
      sc.rho[s] = v;
      break;
    }
    case LSQR_INIT_BETA: {
      const double beta = sqrt(v);
      ls[LS_BETA] = beta;
      ls[LS_PHIBAR] = beta;
      ls[LS_ANORM2] = 0.0;
      ls[LS_RNORM0] = beta;
      ls[LS_TEST] = 1.0;
      sc.its[s] = 0;
      sc.done[s] = !isfinite(v) ? 2 : (beta == 0.0 ? 1 : 0);
      break;
    }
    case LSQR_INIT_ALPHA: {
      if (sc.done[s] != 0) { ls[LS_ALPHA] = 0.0; break; }
      if (!isfinite(v) || v < 0.0) { sc.done[s] = 2; ls[LS_ALPHA] = 0.0; break; }
      const double alpha = sqrt(v);
      ls[LS_ALPHA] = alpha;
      ls[LS_RHOBAR] = alpha;
      if (alpha == 0.0) { sc.done[s] = 1; ls[LS_TEST] = 0.0; }
      break;
    }
    case LSQR_BETA: {
      if (sc.done[s] == 3) sc.done[s] = 1;
      if (sc.done[s] != 0) break;
      if (!isfinite(v)) { sc.done[s] = 2; break; }
      const double beta = sqrt(v);
      const double a = ls[LS_ALPHA];
      ls[LS_ANORM2] += a * a + beta * beta;
      ls[LS_BETA] = beta;
      break;
    }
    case LSQR_ALPHA: {
      if (sc.done[s] != 0) break;
      if (!isfinite(v) || v < 0.0) { sc.done[s] = 2; break; }
      const double alpha = sqrt(v);
      const double rhobar = ls[LS_RHOBAR], beta = ls[LS_BETA], phibar = ls[LS_PHIBAR];
      const double rho = hypot(rhobar, beta);
      const double c = rhobar / rho, sn = beta / rho;
      const double theta = sn * alpha;
      const double phi = c * phibar;
      const double phibar_new = sn * phibar;
      const double tau = sn * phi;
      ls[LS_RHOBAR] = -c * alpha;
      ls[LS_PHIBAR] = phibar_new;
      ls[LS_T1] = phi / rho;
      ls[LS_T2] = -theta / rho;
      ls[LS_ALPHA] = alpha;
      const double anorm = sqrt(ls[LS_ANORM2]);
      const double test = (phibar_new == 0.0) ? 0.0 : alpha * fabs(tau) / (anorm * phibar_new);
      ls[LS_TEST] = test;
      sc.its[s] += 1;
      if (!isfinite(test) || !isfinite(ls[LS_T1])) sc.done[s] = 2;
      else if (test <= R.tol || alpha == 0.0) sc.done[s] = 3;
      break;
    }
  }
}

// A value that workgroups on other XCDs read in the same launch: agent-scope
// accesses, which pass the L2 of the writer's (and the reader's) XCD.
__device__ inline void agent_store(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline double agent_load(const double* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Counts this workgroup in at *cnt after its agent-scope stores have arrived;
// true for the last of nblk, which also resets the count for the next launch.
// One thread calls it.
__device__ inline bool count_in(int32_t* cnt, int nblk) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // the stores this count stands for
  const int before = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (before != nblk - 1) return false;
  __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return true;
}

// The last workgroup of a segment, in two levels: counters of COUNT_GROUP
// workgroups each, then one for the groups, every counter in a cache line of
// its own.  Atomics on one line are served one after the other (about 10 ns
// each): with one counter per segment, side by side, a dot product over 64
// segments of the batch (12,000 workgroups) took 123 us, over one segment of
// 250,000 7.8 us.
__device__ inline bool last_block(int32_t* cnt, int blk, int nblk, int* sh) {
  if (threadIdx.x == 0) {
    const int g = blk / COUNT_GROUP, ng = (nblk + COUNT_GROUP - 1) / COUNT_GROUP;
    bool last = count_in(cnt + (1 + g) * COUNT_STRIDE, min(COUNT_GROUP, nblk - g * COUNT_GROUP));
    if (last && ng > 1) last = count_in(cnt, ng);
    *sh = last;
  }
  __syncthreads();
  return *sh != 0;
}

// Ends a reduction: v, v2 are this workgroup's sums over its chunk of segment
// s.  The last workgroup of the segment adds the chunks (at most RED_BLOCKS,
// one per thread) and takes the step, which spares a launch per reduction:
// the separate kernel that added 256 partial sums in one thread took 5.6 -
// 10 us per call, three calls per CG iteration.  Sums and step together, 250,000
// columns: 4.7 + 5.6 us -> 6.6; with the update of x and r 4.9 + 4.7 + 5.6 ->
// 7.8; 64 segments of 3e6 columns in all: 11.5 + 10.2 -> 15.5 and 33 + 11.5 +
// 10.2 -> 30.
__device__ inline void finish_reduction(const Reduction& R, const Chunk& c, double v, double v2, double* sh) {
  __shared__ int flag;
  const int s = c.seg, nb = c.n, t = threadIdx.x;
  if (nb > 1) {
    double* P = R.partial + (int64_t)s * 2 * RED_BLOCKS;
    if (t == 0) {
      agent_store(P + c.k, v);
      if (R.two) agent_store(P + RED_BLOCKS + c.k, v2);
    }
    if (!last_block(R.count + (int64_t)c.slot * COUNT_LEN, c.k, nb, &flag)) return;
    v = block_reduce_256(t < nb ? agent_load(P + t) : 0.0, sh);
    if (R.two) v2 = block_reduce_256(t < nb ? agent_load(P + RED_BLOCKS + t) : 0.0, sh);
  }
  if (t == 0) reduction_step(R, s, v, v2);
}

// One pass over a segmented vector with a sum: what is done per element, and
// what is summed (v, for RED_DOT2 also v2).
//   RED_DOT:   v = a b
//   RED_DOT2:  v = a b, v2 = c b
//   RED_COPY:  o = b,        v = a b             (p = z, rho = r^T z)
//   RED_START: o = 0, o2 = a, v = a a            (x = 0, r = rhs)
//   RED_SUB:   o = a - b,    v = o o
//   RED_AXPY:  o += f a, o2 -= f b, v = o2 o2    (x, r of a CG step; c, if
//              given, keeps the old o2)
//   RED_LSQR:  o = a - alpha o on active instances (first: o = a), v = o o
// A workgroup takes a chunk; every thread has four elements in flight.
template <int KIND>
__global__ void __launch_bounds__(256)
k_reduce(const Chunk* __restrict__ chunks, RedVec V, Reduction R) {
  __shared__ double sh[4];
  const Chunk c = chunks[blockIdx.x];
  const int s = c.seg;
  const int64_t c0 = c.lo, c1 = c.lo + c.len;
  const double* __restrict__ a = V.a;
  const double* __restrict__ b = V.b;
  double* __restrict__ o = V.o;
  double* __restrict__ o2 = V.o2;
  double f = 0.0;
  bool act = true;
  if constexpr (KIND == RED_AXPY) f = R.sc.alpha[s];
  if constexpr (KIND == RED_LSQR) {
    act = R.sc.done[s] == 0;
    f = V.first ? 0.0 : R.lsqr[(int64_t)s * LSQR_NSC + LS_ALPHA];
  }
  double v = 0.0, v2 = 0.0;
  // U elements 256 apart, all their loads before the first store
  auto elements = [&](int64_t k0, auto uc) {
    constexpr int U = decltype(uc)::value;
    constexpr bool HAS_B = KIND != RED_START && KIND != RED_LSQR;
    constexpr bool HAS_O = KIND == RED_AXPY || KIND == RED_LSQR;
    double ea[U], eb[U], ec[U], eo[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t k = k0 + 256 * u;
      ea[u] = a[k];
      if constexpr (HAS_B) eb[u] = b[k];
      if constexpr (KIND == RED_DOT2) ec[u] = V.c[k];
      if constexpr (KIND == RED_AXPY) ec[u] = o2[k];
      if constexpr (HAS_O) eo[u] = o[k];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t k = k0 + 256 * u;
      if constexpr (KIND == RED_DOT) {
        v += ea[u] * eb[u];
      } else if constexpr (KIND == RED_DOT2) {
        v += ea[u] * eb[u];
        v2 += ec[u] * eb[u];
      } else if constexpr (KIND == RED_COPY) {
        o[k] = eb[u];
        v += ea[u] * eb[u];
      } else if constexpr (KIND == RED_START) {
        o[k] = 0.0;
        o2[k] = ea[u];
        v += ea[u] * ea[u];
      } else if constexpr (KIND == RED_SUB) {
        const double t = ea[u] - eb[u];
        o[k] = t;
        v += t * t;
      } else if constexpr (KIND == RED_AXPY) {
        const double t = ec[u] - f * eb[u];
        o[k] = eo[u] + f * ea[u];
        if (V.keep) V.keep[k] = ec[u];
        o2[k] = t;
        v += t * t;
      } else {
        const double t = !act ? eo[u] : V.first ? ea[u] : ea[u] - f * eo[u];
        o[k] = t;
        v += t * t;
      }
    }
  };
  int64_t k = c0 + threadIdx.x;
  for (; k + 3 * 256 < c1; k += 4 * 256) elements(k, std::integral_constant<int, 4>{});
  for (; k < c1; k += 256) elements(k, std::integral_constant<int, 1>{});
  v = block_reduce_256(v, sh);
  if constexpr (KIND == RED_DOT2) v2 = block_reduce_256(v2, sh);
  finish_reduction(R, c, v, v2, sh);
}

// A segment's chunks: size elements each, at most most of them (then larger ones),
// at least one.  Reductions: 1,024 elements (four per thread), or as many as keep
// the whole vector to RED_TOTAL chunks, and at most RED_BLOCKS per segment, so
// that a long segment gets its workgroups whatever lies beside it: 4,200 segments of
// 32 elements beside one of 1e6 took one workgroup for it when RED_TOTAL was split
// evenly.  A segment of one chunk has no exchange between workgroups.
std::vector<Chunk> make_chunks(const std::vector<int64_t>& seg, int64_t size, int64_t most) {
  std::vector<Chunk> out;
  int32_t slots = 0;
  for (size_t s = 0; s + 1 < seg.size(); ++s) {
    const int64_t len = seg[s + 1] - seg[s];
    const int64_t n = std::max<int64_t>(1, std::min(most, (len + size - 1) / size));
    const int64_t per = (len + n - 1) / n;
    const int32_t slot = n > 1 ? slots++ : 0;
    for (int64_t k = 0; k < n; ++k) {
      const int64_t lo = std::min(len, k * per);
      out.push_back(Chunk{seg[s] + lo, (int32_t)(std::min(len, lo + per) - lo), (int32_t)s, (int32_t)k, (int32_t)n, slot, 0});
    }
  }
  return out;
}

int64_t reduction_chunk(int64_t total) { return std::max<int64_t>(1024, (total + RED_TOTAL - 1) / RED_TOTAL); }

void launch_reduce(hipStream_t st, int kind, const Segments& G, const RedVec& V, const Reduction& R) {
  const unsigned grid = (unsigned)G.red.n;
  const Chunk* c = G.red.c;
  switch (kind) {
    case RED_DOT: k_reduce<RED_DOT><<<grid, 256, 0, st>>>(c, V, R); break;
    case RED_DOT2: k_reduce<RED_DOT2><<<grid, 256, 0, st>>>(c, V, R); break;
    case RED_COPY: k_reduce<RED_COPY><<<grid, 256, 0, st>>>(c, V, R); break;
    case RED_START: k_reduce<RED_START><<<grid, 256, 0, st>>>(c, V, R); break;
    case RED_SUB: k_reduce<RED_SUB><<<grid, 256, 0, st>>>(c, V, R); break;
    case RED_AXPY: k_reduce<RED_AXPY><<<grid, 256, 0, st>>>(c, V, R); break;
    default: k_reduce<RED_LSQR><<<grid, 256, 0, st>>>(c, V, R);
  }
}

__device__ inline int seg_of(int64_t k, int S, const int64_t* seg_ptr) {
  int lo = 0, hi = S - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (seg_ptr[mid] <= k) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// p = z + beta p, a workgroup per piece of up to 1,024 elements
__global__ void __launch_bounds__(256)
k_xpby(const Chunk* __restrict__ fine, const double* __restrict__ beta,
       const double* __restrict__ z, double* __restrict__ p) {
  const Chunk c = fine[blockIdx.x];
  const int64_t k0 = c.lo + threadIdx.x, hi = c.lo + c.len;
  const double b = beta[c.seg];
  double zv[4], pv[4];
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (k0 + 256 * u < hi) {
      zv[u] = z[k0 + 256 * u];
      pv[u] = p[k0 + 256 * u];
    }
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (k0 + 256 * u < hi) p[k0 + 256 * u] = zv[u] + b * pv[u];
}

void launch_xpby(hipStream_t st, const Segments& G, const double* beta, const double* z, double* p) {
  k_xpby<<<(unsigned)G.fine.n, 256, 0, st>>>(G.fine.c, beta, z, p);
}

__global__ void k_sub(int64_t n, const double* __restrict__ a, const double* __restrict__ b,
                      double* __restrict__ out) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) out[k] = a[k] - b[k];
}

void launch_sub(hipStream_t st, int64_t n, const double* a, const double* b, double* out) {
  if (n == 0) return;
  k_sub<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(n, a, b, out);
}

__global__ void k_add(int64_t n, const double* __restrict__ a, const double* __restrict__ b,
                      double* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = a[i] + b[i];
}

void launch_add(hipStream_t st, int64_t n, const double* a, const double* b, double* out) {
  if (n == 0) return;
  k_add<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(n, a, b, out);
}

__global__ void k_fill(int64_t n, double v, double* __restrict__ out) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) out[k] = v;
}

__global__ void k_copy(int64_t n, const double* __restrict__ a, double* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = a[i];
}

void launch_copy(hipStream_t st, int64_t n, const double* a, double* out) {
  if (n == 0) return;
  k_copy<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(n, a, out);
}

void launch_fill(hipStream_t st, int64_t n, double v, double* out) {
  if (n == 0) return;
  k_fill<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(n, v, out);
}

__global__ void k_fill_i32(int64_t n, int32_t v, int32_t* __restrict__ out) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) out[k] = v;
}

void launch_fill_i32(hipStream_t st, int64_t n, int32_t v, int32_t* out) {
  if (n == 0) return;
  k_fill_i32<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(n, v, out);
}

__global__ void k_hash_fill(int64_t n, double* __restrict__ out) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  uint64_t h = (uint64_t)k * 0x9E3779B97F4A7C15ull + 0x632BE59BD9B4E019ull;
  h ^= h >> 31;
  h *= 0xBF58476D1CE4E5B9ull;
  h ^= h >> 29;
  out[k] = (double)(h >> 11) * (2.0 / 9007199254740992.0) - 1.0;
}

void launch_hash_fill(hipStream_t st, int64_t n, double* out) {
  if (n == 0) return;
  k_hash_fill<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(n, out);
}

// ---------------------------------------------------------------------------
// LSQR (Section 4.1, "Solution phase"): Golub-Kahan bidiagonalization of
// A W^{-1}, M = W^{-1} W^{-T}, carried in x-space.  With v the unit vector of
// the bidiagonalization, the iteration keeps vt = W^{-1} v and zh = W^T v:
//   u <- (A vt - alpha u) / beta,
//   q  = A^T u - beta zh,  s = M q,  alpha = sqrt(q^T s),
//   zh <- q / alpha,  vt <- s / alpha,
// so alpha = ||W^{-T} A^T u - beta v|| needs products with M only.  The
// plane rotations, the step x += (phi / rho) wt, wt <- vt - (theta / rho) wt
// and the estimates ||A W^{-1}||_F^2 = sum (alpha^2 + beta^2),
// ||(A W^{-1})^T r|| = alpha |c phibar|-style follow Paige and Saunders.
// done: 0 active, 1 converged, 2 breakdown, 3 converged by this step (its
// update still applies).
// ---------------------------------------------------------------------------
__global__ void k_lsqr_unorm(int64_t m, int S, const int64_t* __restrict__ seg_ptr,
                             const double* __restrict__ sc, const int32_t* __restrict__ done,
                             double* __restrict__ u) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= m) return;
  const int s = S == 1 ? 0 : seg_of(k, S, seg_ptr);
  if (done[s] != 0) return;
  const double beta = sc[(int64_t)s * LSQR_NSC + LS_BETA];
  u[k] = beta > 0.0 ? u[k] / beta : 0.0;
}

void launch_lsqr_unorm(hipStream_t st, int64_t m, int S, const int64_t* seg_row, const double* sc,
                       const int32_t* done, double* u) {
  if (m == 0) return;
  k_lsqr_unorm<<<(unsigned)((m + 255) / 256), 256, 0, st>>>(m, S, seg_row, sc, done, u);
}

__global__ void k_lsqr_q(int64_t n, int S, const int64_t* __restrict__ seg_ptr,
                         const double* __restrict__ sc, const int32_t* __restrict__ done,
                         const double* __restrict__ zh, double* __restrict__ q, int first) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int s = S == 1 ? 0 : seg_of(k, S, seg_ptr);
  if (done[s] != 0) { q[k] = 0.0; return; }
  if (!first) q[k] -= sc[(int64_t)s * LSQR_NSC + LS_BETA] * zh[k];
}

void launch_lsqr_q(hipStream_t st, int64_t n, int S, const int64_t* seg_col, const double* sc,
                   const int32_t* done, const double* zh, double* q, int first) {
  if (n == 0) return;
  k_lsqr_q<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(n, S, seg_col, sc, done, zh, q, first);
}

__global__ void k_lsqr_update(int64_t n, int S, const int64_t* __restrict__ seg_ptr,
                              const double* __restrict__ scb, const int32_t* __restrict__ done,
                              const double* __restrict__ q, const double* __restrict__ sv,
                              double* __restrict__ zh, double* __restrict__ v,
                              double* __restrict__ w, double* __restrict__ x, int first) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int s = S == 1 ? 0 : seg_of(k, S, seg_ptr);
  const int dn = done[s];
  if (!(dn == 0 || dn == 3)) return;
  const double* sc = scb + (int64_t)s * LSQR_NSC;
  const double alpha = sc[LS_ALPHA];
  const double ia = alpha > 0.0 ? 1.0 / alpha : 0.0;
  const double vn = sv[k] * ia;
  zh[k] = q[k] * ia;
  v[k] = vn;
  if (first) {
    w[k] = vn;
  } else {
    const double wo = w[k];
    x[k] += sc[LS_T1] * wo;
    w[k] = vn + sc[LS_T2] * wo;
  }
}

void launch_lsqr_update(hipStream_t st, int64_t n, int S, const int64_t* seg_col, const double* sc,
                        const int32_t* done, const double* q, const double* s, double* zh,
                        double* v, double* w, double* x, int first) {
  if (n == 0) return;
  k_lsqr_update<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(n, S, seg_col, sc, done, q, s, zh, v,
                                                             w, x, first);
}

// ---------------------------------------------------------------------------
// GMRES building blocks: Gram-Schmidt against the stored basis V, with
// per-instance coefficients and fixed-order reductions
// ---------------------------------------------------------------------------
// h[s ld + i] = V_i . w over segment s, i < kv, eight vectors per workgroup so
// that w is read once for them; chunk sums go through partial (MDOT_BLOCKS per
// vector), added by the last workgroup of the eight.  sum, if given, also
// takes h (the total over the two passes of Gram-Schmidt).  One vector after
// the other with a barrier each, and one thread per vector adding 256 partial
// sums, took 13.4 + 16.5 us per pass (mean over 1 to 30 vectors of 90,601); this
// takes 7.5.
// Its segments have at most 64 chunks: the groups of eight vectors fill the chip too.
__global__ void __launch_bounds__(256)
k_multidot(const Chunk* __restrict__ chunks, int64_t n, int kv, const double* __restrict__ V,
           const double* __restrict__ w, double* __restrict__ partial, int32_t* __restrict__ count,
           int ld, double* __restrict__ h, double* __restrict__ sum) {
  __shared__ double sh[4][MDOT];
  __shared__ int flag;
  const Chunk ch = chunks[blockIdx.x];
  const int s = ch.seg, i0 = blockIdx.y * MDOT, nv = min(MDOT, kv - i0), nb = ch.n;
  const int t = threadIdx.x, lane = t % 64, wave = t / 64;
  const int64_t c0 = ch.lo, c1 = ch.lo + ch.len;
  const double* v[MDOT];
  double acc[MDOT];
#pragma unroll
  for (int i = 0; i < MDOT; ++i) {
    v[i] = V + (int64_t)(i0 + min(i, nv - 1)) * n;
    acc[i] = 0.0;
  }
  for (int64_t k = c0 + t; k < c1; k += 256) {
    const double x = w[k];
#pragma unroll
    for (int i = 0; i < MDOT; ++i) acc[i] += v[i][k] * x;
  }
#pragma unroll
  for (int i = 0; i < MDOT; ++i) {
    acc[i] = wave_allsum(acc[i]);
    if (lane == 0) sh[wave][i] = acc[i];
  }
  __syncthreads();
  double* P = partial + ((int64_t)s * ld + i0) * MDOT_BLOCKS;
  if (wave == 0) {
    if (lane < nv)
      agent_store(P + (int64_t)lane * MDOT_BLOCKS + ch.k,
                  (sh[0][lane] + sh[1][lane]) + (sh[2][lane] + sh[3][lane]));
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // all lanes' stores, before the count
  }
  if (t == 0) flag = count_in(count + ((int64_t)s * gridDim.y + blockIdx.y) * COUNT_STRIDE, nb);
  __syncthreads();
  if (!flag) return;
  for (int i = wave; i < nv; i += 4) {
    const double x = wave_allsum(lane < nb ? agent_load(P + (int64_t)i * MDOT_BLOCKS + lane) : 0.0);
    if (lane == 0) {
      h[(int64_t)s * ld + i0 + i] = x;
      if (sum) sum[(int64_t)s * ld + i0 + i] += x;
    }
  }
}

void launch_multidot(hipStream_t st, const Segments& G, int64_t n, int k, const double* V,
                     const double* w, double* partial, int32_t* count, int ld, double* h,
                     double* sum) {
  if (k == 0) return;
  const dim3 grid((unsigned)G.mdot.n, (k + MDOT - 1) / MDOT);
  k_multidot<<<grid, 256, 0, st>>>(G.mdot.c, n, k, V, w, partial, count, ld, h, sum);
}

// out_k (-)= sum_i V_i[k] c[seg(k) * ld + i]
template <bool SUB>
__global__ void k_multi_comb(int S, const int64_t* __restrict__ seg_ptr, int64_t n, int kv,
                             const double* __restrict__ V, const double* __restrict__ c, int ld,
                             double* __restrict__ out) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int s = S == 1 ? 0 : seg_of(k, S, seg_ptr);
  const double* cs = c + (int64_t)s * ld;
  double acc = 0.0;
#pragma unroll 8
  for (int i = 0; i < kv; ++i) acc += V[(int64_t)i * n + k] * cs[i];
  out[k] = SUB ? out[k] - acc : acc;
}

void launch_multi_axpy(hipStream_t st, int S, const int64_t* seg_ptr, int64_t n, int k,
                       const double* V, const double* h, int ld, double* w) {
  if (n == 0 || k == 0) return;
  k_multi_comb<true><<<(unsigned)((n + 255) / 256), 256, 0, st>>>(S, seg_ptr, n, k, V, h, ld, w);
}

void launch_multi_gemv(hipStream_t st, int S, const int64_t* seg_ptr, int64_t n, int k,
                       const double* V, const double* y, int ld, double* out) {
  if (n == 0) return;
  k_multi_comb<false><<<(unsigned)((n + 255) / 256), 256, 0, st>>>(S, seg_ptr, n, k, V, y, ld, out);
}

__global__ void k_normalize_seg(int64_t n, int S, const int64_t* __restrict__ seg_ptr,
                                const double* __restrict__ nrm2, const int32_t* __restrict__ done,
                                const double* __restrict__ a, double* __restrict__ out) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int s = S == 1 ? 0 : seg_of(k, S, seg_ptr);
  const double q = nrm2[s];
  const bool ok = q > 0.0 && isfinite(q) && (done == nullptr || done[s] == 0);
  out[k] = ok ? a[k] / sqrt(q) : 0.0;
}

void launch_normalize_seg(hipStream_t st, int64_t n, int S, const int64_t* seg_ptr,
                          const double* nrm2, const int32_t* done, const double* a, double* out) {
  if (n == 0) return;
  k_normalize_seg<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(n, S, seg_ptr, nrm2, done, a, out);
}

}  // namespace lsq2l
