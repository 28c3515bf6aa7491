// Per-iteration local solves of the preconditioner: C_ii^{-1} R_i r for every
// subdomain with its factor L L^T (Algorithm 1, the local terms of
// eq. (two_level_schwarz)), with FP64 or FP32 factors.
//
// The factors come as 32 x 32 tile envelopes with inverted diagonal tiles
// D_I = L_II^{-1}.  What an application reads is a copy laid out for it once
// per setup, per subdomain:
//   * the packed D_I: the ten 8 x 8 blocks of its lower triangle;
//   * the forward stream, rows of M = D L (M_I = D_I L(I, :) left of the
//     diagonal tile), and the backward stream, rows of P^T, P = L D
//     (P(K, I) = L(K, I) D_I).
// With t = D b, L y = b is y_I = t_I - sum_J M(I, J) y_J, and with t' = D^T y,
// L^T x = y is x_I = t'_I - sum_K P(K, I)^T x_K: both products with D are
// independent over the rows and leave one product with the previous block on
// the chain of dependent steps, where the plain substitution has a second
// one, with D_I, after it.  The streams keep the columns of a row that its
// entries reach in groups of eight ("slabs", 32 x 8) instead of whole tiles:
// on a band of half-width 40 an application reads 3,840 entries per 32
// unknowns, where tiles and inverses read 6,144.
#include <algorithm>

#include "kernels.hpp"

namespace lsq2l {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
template <typename T> struct StreamCfg;
template <> struct StreamCfg<float> {
  using V = f32x4;
  static constexpr int DC = 4, DH = 12;      // chain tiles / slabs of a wave in flight
};
template <> struct StreamCfg<double> {
  using V = f64x2;
  static constexpr int DC = 2, DH = 8;
};
// A stream is read in 16-byte vectors of VE entries of one column; the lanes
// of a wave form NG groups that hold the 32 rows of a column each.
template <typename T> struct StreamMap {
  static constexpr int VE = 16 / sizeof(T);
  static constexpr int NG = 2 * VE;          // 64 lanes / (32 / VE)
  static constexpr int CC = TS / NG;         // columns of a chain tile per lane
  static constexpr int CS = 8 / NG;          // columns of a slab per lane
  // place of entry (r, c) in a chain tile (32 x 32) and in a slab (32 x 8):
  // vector i of the lane in group g holds column CC g + i (CS g + i)
  __host__ __device__ static int chain_at(int r, int c) { return (c % CC) * (64 * VE) + (c / CC) * TS + r; }
  __host__ __device__ static int slab_at(int r, int c) { return (c % CS) * (64 * VE) + (c / CS) * TS + r; }
};
constexpr int SLAB = TS * 8;
constexpr int SOLVE_WAVES = 8;
constexpr int CHAIN = 2;                     // waves that take the chain tiles in turn
constexpr int HELPERS = SOLVE_WAVES - CHAIN; // waves that take the slabs
constexpr int DPACK = SOLVE_DPACK;           // entries of a packed D_I: ten 8 x 8 blocks
static_assert(SOLVE_FAR_INTS == 2 * (HELPERS + 1), "far0 entries");
// Largest subdomain that the streams solve; larger ones are solved in global
// memory (k_local_solve).  FP64 factors: where the local vector fits in LDS beside
// the tables (148 of 160 KB).  FP32 factors: 12,544 unknowns.  The streams hold
// the vector and its sums in the factors' type, k_local_solve holds them in double:
// M r on one banded subdomain of 13,000 / 18,944 unknowns is off by 1.15e-7 /
// 1.24e-7 with it, by 1.27e-7 / 1.42e-7 with streams (which take 0.30 / 0.43 ms
// instead of 1.4 / 2.4).
template <typename T> constexpr int SCAP_OF = sizeof(T) == 8 ? 18944 : 12544;
constexpr int SCAP = SCAP_OF<double>;
constexpr int SCAP_TILES = SCAP / TS;

// x + x of the lane 8 / 16 away within its row of 16 / pair of rows
__device__ inline double ror8_sum(double x) { return dpp_pair_sum<0x128>(x); }
__device__ inline float ror8_sum(float x) {
  return x + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x128, 0xF, 0xF, false));
}
__device__ inline float row16_pair_sum(float x) {
  const int v = __float_as_int(x);
  const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  return __int_as_float(r[0]) + __int_as_float(r[1]);
}
__device__ inline double row16_pair_sum(double x) {
  const int lo = __double2loint(x), hi = __double2hiint(x);
  const auto rlo = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
  const auto rhi = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
  return __hiloint2double(rhi[0], rlo[0]) + __hiloint2double(rhi[1], rlo[1]);
}
// sum over the NG lane groups of a stream vector
__device__ inline double group_sum(double x) { return half_pair_sum(row16_pair_sum(x)); }
__device__ inline float group_sum(float x) { return half_pair_sum(row16_pair_sum(ror8_sum(x))); }
// sum over the eight lanes of an aligned group, and over the groups
__device__ inline double oct_sum(double x) {
  return dpp_pair_sum<0x141>(dpp_pair_sum<0x4E>(dpp_pair_sum<0xB1>(x)));
}
__device__ inline float oct_sum(float x) {
  x += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0xB1, 0xF, 0xF, false));
  x += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x4E, 0xF, 0xF, false));
  return x + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x141, 0xF, 0xF, false));
}
template <typename T>
__device__ inline T across_octs_sum(T x) { return half_pair_sum(row16_pair_sum(ror8_sum(x))); }

// ---------------------------------------------------------------------------
// layout of the streams
// ---------------------------------------------------------------------------
// Step s of the forward sweep handles block row s, of the backward sweep
// block nt - 1 - s.  Chain tile s is the block coupled to the previous step's
// result; the slabs of the step are its further columns in ascending order,
// slab j going to helper j % HELPERS, whose slabs of all steps lie one after
// the other.  Per subdomain and sweep, the stream is nt chain tiles and then
// the helpers' slabs: at most as many entries as the subdomain's envelope
// (nt diagonal tiles and the rest), so it starts at fac_off.
// f8[g] = first column any of the rows 8 g .. 8 g + 7 reaches.
__global__ void __launch_bounds__(256)
k_stream_layout(const SubDesc* __restrict__ subs, const int32_t* __restrict__ tileF,
                const int64_t* __restrict__ tileOff, const int32_t* __restrict__ F8,
                const SubDesc* __restrict__ gsub, SolveStream S) {
  __shared__ int f8[4 * SCAP_TILES];
  __shared__ int cnt[SCAP_TILES], off[HELPERS][SCAP_TILES], wb[HELPERS + 1];
  const SubDesc d = subs[blockIdx.x];
  if (d.np > S.cap) return;
  const int nt = d.ntiles, tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
  const int32_t* F = tileF + d.tile_base;
  const int64_t* O = tileOff + d.tile_base;
  const int32_t* own = d.spare ? F8 + 4 * gsub[d.id].tile_base : nullptr;
  for (int g = tid; g < 4 * nt; g += 256) f8[g] = own ? own[g] : TS * F[g / 4];
  __syncthreads();
  const int64_t tile0 = d.fac_off / TT, slab0 = d.fac_off / SLAB;
  auto first8 = [&](int I) {
    return min(min(f8[4 * I], f8[4 * I + 1]), min(f8[4 * I + 2], f8[4 * I + 3])) / 8;
  };
  for (int dir = 0; dir < 2; ++dir) {
    uint16_t* nf = S.nfar[dir] + d.tile_base;
    int32_t* pos = S.pos[dir] + 4 * tile0;
    int32_t* desc = S.desc[dir] + slab0;
    if (dir == 0) {
      for (int s = tid; s < nt; s += 256) cnt[s] = s ? max(0, 4 * (s - 1) - first8(s)) : 0;
    } else {
      for (int s = wave; s < nt; s += 4) {
        const int J = nt - 1 - s;
        int c = 0;
        for (int g0 = 4 * (J + 2); g0 < 4 * nt; g0 += 64)
          c += __popcll(__ballot(g0 + lane < 4 * nt && f8[min(g0 + lane, 4 * nt - 1)] < TS * (J + 1)));
        if (lane == 0) cnt[s] = c;
      }
    }
    __syncthreads();
    for (int s = tid; s < nt; s += 256) nf[s] = (uint16_t)cnt[s];
    if (tid < HELPERS) {
      int run = 0;
      for (int s = 0; s < nt; ++s) {
        off[tid][s] = run;
        run += (cnt[s] + HELPERS - 1 - tid) / HELPERS;
      }
      wb[tid + 1] = run;
    }
    __syncthreads();
    if (tid == 0) {
      wb[0] = 0;
      for (int w = 0; w < HELPERS; ++w) wb[w + 1] += wb[w];
      for (int w = 0; w <= HELPERS; ++w) S.far0[(d.id * 2 + dir) * (HELPERS + 1) + w] = wb[w];
    }
    __syncthreads();
    for (int s = wave; s < nt; s += 4) {
      auto place = [&](int j, int group, int K, int J) {   // slab j of step s: rows / columns 8 group ..
        const int w = j % HELPERS, at = wb[w] + off[w][s] + j / HELPERS;
        pos[4 * (O[K] + (J - F[K])) + group % 4] = at;
        desc[at] = group;
      };
      if (dir == 0) {
        const int g = first8(s);
        for (int j = lane; j < cnt[s]; j += 64) place(j, g + j, s, (g + j) / 4);
      } else {
        const int J = nt - 1 - s;
        int before = 0;
        for (int g0 = 4 * (J + 2); g0 < 4 * nt; g0 += 64) {
          const int g = g0 + lane;
          const bool hit = g < 4 * nt && f8[min(g, 4 * nt - 1)] < TS * (J + 1);
          const unsigned long long m = __ballot(hit);
          if (hit) place(before + __popcll(m & ((1ull << lane) - 1ull)), g, g / 4, J);
          before += __popcll(m);
        }
      }
    }
    __syncthreads();
  }
}

// The streams' entries from a factor: wave by wave over the tile rows K of a
// subdomain, the packed D_K and, per tile (K, J), M(K, J) and P(K, J) as 16 x 16
// MFMA blocks, formed so that the rows of a stored column lie on consecutive
// lanes.  Operands read across columns are staged in LDS.  On wide envelopes it
// takes several times what the factor read once and the streams written once
// would (512 irregular subdomains 3.7 ms in FP64, 7.8 in FP32 beside the
// selection): tile after tile, a wave waits for two operands, forms two products
// and stores them 16 rows of a column at a time.  64 banded problems 1.6 ms.
template <typename T>
__global__ void __launch_bounds__(256, 2)
k_stream_pack(const SubDesc* __restrict__ subs, const int32_t* __restrict__ tileF,
              const int64_t* __restrict__ tileOff, const T* __restrict__ fac,
              const T* __restrict__ dinv, SolveStream S, T* __restrict__ fwd, T* __restrict__ bwd,
              T* __restrict__ dpack) {
  using Map = StreamMap<T>;
  __shared__ T sL[4][TS * LDT], sD[4][TS * LDT];
  const SubDesc d = subs[blockIdx.x];
  if (d.np > S.cap) return;
  const int nt = d.ntiles, lane = threadIdx.x % 64;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int li = lane % 16, lk = lane / 16;
  const int32_t* F = tileF + d.tile_base;
  const int64_t* O = tileOff + d.tile_base;
  const T* A = fac + d.fac_off;
  const T* Di = dinv + d.dinv_off;
  for (int K = blockIdx.y * 4 + wave; K < nt; K += 4 * gridDim.y) {
    const T* DK = Di + (int64_t)K * TT;
    T* dp = dpack + d.dinv_off / TT * DPACK + (int64_t)K * DPACK;
#pragma unroll
    for (int bi = 0; bi < 4; ++bi)
#pragma unroll
      for (int bj = 0; bj <= bi; ++bj)
        dp[(bi * (bi + 1) / 2 + bj) * 64 + lane] = DK[(8 * bj + lane / 8) * TS + 8 * bi + lane % 8];
    const int f = F[K];
    if (K > 0 && f == K)                        // not coupled to the previous block
      for (int e = lane; e < TT; e += 64) {
        fwd[d.fac_off + (int64_t)K * TT + e] = T(0);
        bwd[d.fac_off + (int64_t)(nt - K) * TT + e] = T(0);
      }
    for (int J = f; J < K; ++J) {
      const int64_t t = O[K] + (J - f);
      const T* L = A + t * TT;
      const T* DJ = Di + (int64_t)J * TT;
      T* l = sL[wave];
      T* dj = sD[wave];
      wave_sync();
#pragma unroll
      for (int q = 0; q < TT / 64; ++q) {
        const int e = 64 * q + lane;
        l[(e / TS) * LDT + e % TS] = L[e];
        dj[(e / TS) * LDT + e % TS] = DJ[e];
      }
      wave_sync();
#pragma unroll
      for (int dir = 0; dir < 2; ++dir) {
        // dir 0: acc(c, r) = M(K, J)(r, c) = sum_k D_K(r, k) L(k, c)
        // dir 1: acc(r, c) = P(K, J)(r, c) = sum_k L(r, k) D_J(k, c)
        typename Mfma<T>::acc_t acc[4];
        tile_acc_zero<T>(acc);
#pragma unroll 4
        for (int q = 0; q < 8; ++q) {
          const int k = 4 * q + lk;
          T a[2], b[2];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int i = 16 * h + li;
            a[h] = dir == 0 ? l[i * LDT + k] : l[k * LDT + i];
            b[h] = dir == 0 ? DK[k * TS + i] : dj[i * LDT + k];
          }
#pragma unroll
          for (int h = 0; h < 4; ++h) acc[h] = Mfma<T>::mma(a[h / 2], b[h % 2], acc[h]);
        }
        const bool chain = K == J + 1;
        const int32_t* pp = S.pos[dir] + 4 * (d.fac_off / TT + t);
        const int at0 = pp[0], at1 = pp[1], at2 = pp[2], at3 = pp[3];
        const int step = dir == 0 ? K : nt - 1 - J;
        T* out = (dir == 0 ? fwd : bwd) + d.fac_off + (int64_t)(chain ? step : nt) * TT;
#pragma unroll
        for (int h = 0; h < 4; ++h)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            // stored row sr, stored column sc of the product
            const int sr = 16 * (h % 2) + Mfma<T>::acc_col(lane, v);
            const int sc = 16 * (h / 2) + Mfma<T>::acc_row(lane, v);
            const int u = sc / 8, at = u < 2 ? (u == 0 ? at0 : at1) : (u == 2 ? at2 : at3);
            const int off = chain ? Map::chain_at(sr, sc) : at * SLAB + Map::slab_at(sr, sc % 8);
            if (chain || at >= 0) out[off] = acc[h][v];
          }
      }
    }
  }
}

// scol / sscale: global column and scaling of every position of the layout
// (-1 on padding), so that an application gathers R_i r itself
__global__ void __launch_bounds__(256)
k_solve_cols(const SubDesc* __restrict__ subs, const SubDesc* __restrict__ lay,
             const int32_t* __restrict__ omega, const double* __restrict__ scale,
             const int32_t* __restrict__ sperm, int32_t* __restrict__ scol,
             double* __restrict__ sscale) {
  const SubDesc d = subs[blockIdx.x];
  const SubDesc s = lay[d.id];
  const int32_t* om = omega + d.omega_off;
  for (int q = threadIdx.x; q < s.np; q += blockDim.x) {
    const int64_t at = sperm ? sperm[s.loc_off + q] : d.loc_off + q;
    const int pos = at >= 0 ? (int)(at - d.loc_off) : -1;
    int c = -1;
    if (pos >= 0 && pos < d.nI) c = om[pos];
    else if (pos >= d.nIp && pos < d.nIp + d.nG) c = om[d.nI + pos - d.nIp];
    scol[s.loc_off + q] = c;
    sscale[s.loc_off + q] = c >= 0 ? scale[at] : 0.0;
  }
}

// ---------------------------------------------------------------------------
// the application
// ---------------------------------------------------------------------------
// y_I <- D_I y_I (TRANS: D_I^T y_I) for every block, each by one wave: lane
// (r, c) = (l % 8, l / 8) holds entry (r, c) of every 8 x 8 block.
template <typename T, bool TRANS>
__device__ inline void stream_diag(const T* __restrict__ dp, T* y, int nt, int wave, int lane) {
  constexpr int U = 2;                         // blocks in flight
  T ring[U][10];
  auto load = [&](T (&a)[10], int I) {
    const T* p = dp + (int64_t)min(I, nt - 1) * DPACK + lane;
#pragma unroll
    for (int b = 0; b < 10; ++b) a[b] = p[64 * b];
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int u = 0; u < U; ++u) load(ring[u], wave + SOLVE_WAVES * u);
  for (int I0 = wave; I0 < nt; I0 += SOLVE_WAVES * U) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int I = I0 + SOLVE_WAVES * u;
      if (I < nt) {
        T v[4], o[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          v[q] = y[I * TS + 8 * q + (TRANS ? lane % 8 : lane / 8)];
          o[q] = T(0);
        }
        int b = 0;
#pragma unroll
        for (int bi = 0; bi < 4; ++bi)
#pragma unroll
          for (int bj = 0; bj <= bi; ++bj, ++b) o[TRANS ? bj : bi] += ring[u][b] * v[TRANS ? bi : bj];
#pragma unroll
        for (int q = 0; q < 4; ++q) o[q] = TRANS ? oct_sum(o[q]) : across_octs_sum(o[q]);
        // block row q of the result is taken from the lanes of the other index q
        const int q = TRANS ? lane % 8 : lane / 8;
        const T r = q == 0 ? o[0] : q == 1 ? o[1] : q == 2 ? o[2] : o[3];
        wave_sync();
        if (q < 4) y[I * TS + 8 * q + (TRANS ? lane / 8 : lane % 8)] = r;
        wave_sync();
      }
      __builtin_amdgcn_sched_barrier(0);
      load(ring[u], I + SOLVE_WAVES * U);
    }
  }
}

// One sweep, a barrier per step.  Waves 0 and 1 take the chain tiles in turn,
// from registers filled DC of their steps ahead: together they cover the memory
// latency with few enough registers (128) for two workgroups on a CU, which
// the many small subdomains of the 500 x 500 grid need (62 us per application
// with five tiles per wave and one workgroup, 54 with two tiles).  The other
// waves sum the
// slabs of the following step, whose operands are one step older, and hand
// their sums over in LDS, double buffered; the LDS reads of a slab's operands
// are issued one slab ahead.  The loads of a register slot are issued in one
// order only, on every path and fenced against the scheduler: the compiler
// waits for a slot by counting the loads after it, and with a branch around a
// load, or two orders that meet, it waits for all.
template <typename T, bool REV>
__device__ inline void stream_sweep(const T* __restrict__ stream, const int32_t* __restrict__ desc,
                                    const int32_t* __restrict__ far0, const uint16_t* nf, T* y, T* part,
                                    int nt, int wave, int lane) {
  using V = typename StreamCfg<T>::V;
  using GV = const __attribute__((address_space(1))) V;
  using GB = const __attribute__((address_space(1))) char;
  using GI = const __attribute__((address_space(1))) int32_t;
  using Map = StreamMap<T>;
  constexpr int VE = Map::VE, DC = StreamCfg<T>::DC, DH = StreamCfg<T>::DH;
  constexpr int CV = TT / (64 * VE), SV = SLAB / (64 * VE);     // vectors per lane of a tile / slab
  const int rl = VE * (lane % (TS / VE)), g = lane / (TS / VE);  // first row and group of the lane
  // helpers with any slab at all (a step's first slabs go to the first ones)
  int active = 0;
#pragma unroll
  for (int h = 0; h < HELPERS; ++h) active += far0[h + 1] > far0[h];
  active = __builtin_amdgcn_readfirstlane(active);
  if (wave >= CHAIN)
    for (int r = lane; r < TS; r += 64) part[(HELPERS + wave - CHAIN) * TS + r] = T(0);   // step 1 has no slabs
  __syncthreads();
  if (wave < CHAIN) {
    GB* src = (GB*)stream;
    V ring[DC][CV];
    auto load = [&](V (&a)[CV], int s) {
      GB* at = src + (uint32_t)(min(s, nt - 1) * (TT * (int)sizeof(T)) + 16 * lane);
#pragma unroll
      for (int c = 0; c < CV; ++c) a[c] = *(GV*)(at + 1024 * c);
      __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int i = 0; i < DC; ++i) load(ring[i], 1 + wave + CHAIN * i);
    for (int s0 = 1; s0 < nt; s0 += CHAIN * DC) {
#pragma unroll
      for (int i = 0; i < DC; ++i) {
        const int s = s0 + CHAIN * i + wave;
        for (int j = 0; j < wave; ++j)
          if (s - wave + j < nt) __syncthreads();
        if (s < nt) {
          const int b = REV ? nt - 1 - s : s, pv = REV ? b + 1 : b - 1;
          T* yb = y + b * TS + rl;
          T yc[CV];
#pragma unroll
          for (int c = 0; c < CV / VE; ++c) {
            const V w = reinterpret_cast<const V*>(y + pv * TS + Map::CC * g)[c];
#pragma unroll
            for (int e = 0; e < VE; ++e) yc[c * VE + e] = w[e];
          }
          V t = *reinterpret_cast<const V*>(yb);
          const T* ps = part + (s & 1) * (HELPERS * TS) + rl;
          if (active > 0) {
            V p[HELPERS];
#pragma unroll
            for (int h = 0; h < 2; ++h) p[h] = *reinterpret_cast<const V*>(ps + h * TS);
            if (active > 2) {
#pragma unroll
              for (int h = 2; h < HELPERS; ++h) p[h] = *reinterpret_cast<const V*>(ps + h * TS);
              t -= (p[2] + p[3]) + (p[4] + p[5]);
            }
            t -= p[0] + p[1];
          }
          V a0 = ring[i][0] * yc[0], a1 = ring[i][1] * yc[1];
#pragma unroll
          for (int c = 2; c < CV; c += 2) {
            a0 += ring[i][c] * yc[c];
            a1 += ring[i][c + 1] * yc[c + 1];
          }
          a0 += a1;
#pragma unroll
          for (int e = 0; e < VE; ++e) t[e] -= group_sum(a0[e]);
          if (g == 0) *reinterpret_cast<V*>(yb) = t;
          __syncthreads();
        }
        for (int j = wave + 1; j < CHAIN; ++j)
          if (s - wave + j < nt) __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        load(ring[i], s + CHAIN * DC);
      }
    }
  } else {
    const int h = wave - CHAIN, total = far0[h + 1] - far0[h];
    if (total == 0) {
      for (int r = lane; r < TS; r += 64) part[h * TS + r] = T(0);
      for (int s = 1; s < nt; ++s) __syncthreads();
    } else {
      GB* src = (GB*)(stream + (int64_t)nt * TT + (int64_t)far0[h] * SLAB);
      GI* dsc = (GI*)(desc + far0[h]);
      V ring[DH][SV];
      int grp[DH];
      int k = 0;                                   // next slab to load
      auto load = [&](int i) {
        const int kk = min(k, total - 1);
        GB* at = src + (uint32_t)(kk * (SLAB * (int)sizeof(T)) + 16 * lane);
        grp[i] = dsc[kk];
#pragma unroll
        for (int c = 0; c < SV; ++c) ring[i][c] = *(GV*)(at + 1024 * c);
        ++k;
        __builtin_amdgcn_sched_barrier(0);
      };
#pragma unroll
      for (int i = 0; i < DH; ++i) load(i);
      // slabs of this wave in step s; the table is read a step before the value
      // is needed
      auto entry = [&](int s) { return s < nt ? (int)nf[s] : 0; };
      auto count = [&](int e) { return (int)((unsigned)__builtin_amdgcn_readfirstlane(e + HELPERS - 1 - h) / HELPERS); };
      V acc;
#pragma unroll
      for (int e = 0; e < VE; ++e) acc[e] = T(0);
      int s = 1, left = count(entry(2)), next = entry(3);
      // hands over the sums of step s + 1 while they are complete
      auto finish = [&]() {
        while (left == 0 && s < nt) {
          if (s + 1 < nt) {
#pragma unroll
            for (int e = 0; e < VE; ++e) acc[e] = group_sum(acc[e]);
            if (g == 0) *reinterpret_cast<V*>(part + (((s + 1) & 1) * HELPERS + h) * TS + rl) = acc;
#pragma unroll
            for (int e = 0; e < VE; ++e) acc[e] = T(0);
          }
          __syncthreads();
          ++s;
          left = count(next);
          next = entry(s + 2);
        }
      };
      // N slabs from slot i on, all of one step: the reads of their operands
      // overlap (one slab at a time left each waiting for its own)
      auto consume = [&](int i, auto nc) {
        constexpr int N = decltype(nc)::value;
        T v[N][SV];
#pragma unroll
        for (int u = 0; u < N; ++u) {
          const T* yg = y + 8 * grp[i + u] + Map::CS * g;
#pragma unroll
          for (int c = 0; c < SV; ++c) v[u][c] = yg[c];
        }
#pragma unroll
        for (int u = 0; u < N; ++u)
#pragma unroll
          for (int c = 0; c < SV; ++c) acc += ring[i + u][c] * v[u][c];
        left -= N;
      };
      while (s < nt) {
#pragma unroll
        for (int i = 0; i < DH; i += 4) {
          finish();
          if (left >= 4) {
            consume(i, std::integral_constant<int, 4>{});
          } else if (s < nt) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              finish();
              if (s < nt) consume(i + u, std::integral_constant<int, 1>{});
            }
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int u = 0; u < 4; ++u) load(i + u);
        }
      }
    }
  }
  __syncthreads();
}

// Workgroup b solves subdomain subs[b] (decreasing size) with its local vector
// in LDS: loc(position) = S C_ii^{-1} S r on the positions of Omega_i, S the
// equilibration, which the gather and the result carry.
//
// What bounds it: HBM, at 5.2 - 5.9 TB/s (a copy reaches 4.8) where the
// subdomains are many and alike; else the largest one, whose steps take about
// 0.45 us (a barrier and two rounds through LDS) and whose CU draws at most
// about 45 GB/s.  Against tiles streamed through LDS to one consuming wave,
// gather launch included, per application: 64 banded problems of 3e6 columns
// 0.90 -> 0.60 ms (FP32 factors 0.69 -> 0.46), 1000 x 1000 grid 0.37 -> 0.27,
// 500 x 500 grid 0.088 -> 0.054, 128 irregular subdomains 0.47 -> 0.35.
template <typename T>
__global__ void __launch_bounds__(64 * SOLVE_WAVES, 4)
k_local_solve_stream(const SubDesc* __restrict__ subs, SolveStream S, const T* __restrict__ fwd,
                     const T* __restrict__ bwd, const T* __restrict__ dpack,
                     const double* __restrict__ r, double* __restrict__ loc,
                     const int32_t* __restrict__ sperm) {
  extern __shared__ __align__(16) unsigned char smem[];
  const SubDesc d = subs[blockIdx.x];
  if (d.np > S.cap) return;                       // k_local_solve
  const int nt = d.ntiles, tid = threadIdx.x, lane = tid % 64;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  T* y = reinterpret_cast<T*>(smem);
  T* part = y + d.np;
  uint16_t* nf = reinterpret_cast<uint16_t*>(part + 2 * HELPERS * TS);
  const int32_t* col = S.scol + d.loc_off;
  const double* sc = S.sscale + d.loc_off;
  for (int q = tid; q < d.np; q += 64 * SOLVE_WAVES) {
    const int c = col[q];
    y[q] = c >= 0 ? (T)(sc[q] * r[c]) : T(0);
  }
  for (int s = tid; s < nt; s += 64 * SOLVE_WAVES) {
    nf[s] = S.nfar[0][d.tile_base + s];
    nf[nt + s] = S.nfar[1][d.tile_base + s];
  }
  __syncthreads();
  const T* dp = dpack + d.dinv_off / TT * DPACK;
  const int64_t slab0 = d.fac_off / SLAB;
  const int32_t* far0 = S.far0 + d.id * 2 * (HELPERS + 1);
  stream_diag<T, false>(dp, y, nt, wave, lane);
  stream_sweep<T, false>(fwd + d.fac_off, S.desc[0] + slab0, far0, nf, y, part, nt, wave, lane);
  stream_diag<T, true>(dp, y, nt, wave, lane);
  stream_sweep<T, true>(bwd + d.fac_off, S.desc[1] + slab0, far0 + HELPERS + 1, nf + nt, y, part, nt,
                        wave, lane);
  for (int q = tid; q < d.np; q += 64 * SOLVE_WAVES) {
    const int64_t ix = sperm ? (int64_t)sperm[d.loc_off + q] : d.loc_off + q;
    if (ix >= 0) loc[ix] = sc[q] * (double)y[q];
  }
}

static size_t stream_lds_bytes(int np, size_t elem) {
  return (size_t)np * elem + 2 * HELPERS * TS * elem + 2 * (size_t)(np / TS) * sizeof(uint16_t);
}
static_assert(SCAP * 8 + 2 * HELPERS * TS * 8 + 2 * SCAP_TILES * 2 <= 160 * 1024, "LDS of the local solve");

// Subdomains of above lo and up to hi local unknowns: forward and backward
// substitution by tile rows with y in global memory (with IN_LDS, for handles
// without streams, in LDS), workgroup per subdomain, 32 rows of
// threads each summing every eighth tile of a row (fixed order), the
// diagonal blocks applied through their inverses.
template <typename T, bool IN_LDS>
__global__ void __launch_bounds__(256)
k_local_solve(const SubDesc* __restrict__ subs, const int32_t* __restrict__ tileF,
              const int64_t* __restrict__ tileOff, const T* __restrict__ fac,
              const T* __restrict__ dinv, SolveStream S, const double* __restrict__ rhs,
              double* __restrict__ loc, const int32_t* __restrict__ sperm,
              double* __restrict__ scratch, int lo, int hi) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double part[8][TS];
  __shared__ double sv[TS];
  const SubDesc d = subs[blockIdx.x];
  const int32_t* F = tileF + d.tile_base;
  const int64_t* off = tileOff + d.tile_base;
  const T* A = fac + d.fac_off;
  const T* Di = dinv + d.dinv_off;
  if (d.np <= lo || d.np > hi) return;
  const int32_t* sp = sperm ? sperm + d.loc_off : nullptr;
  // y in global memory: in place in loc, or, for a permuted layout, in the
  // subdomain's slice of scratch
  double* y;
  if constexpr (IN_LDS) y = reinterpret_cast<double*>(smem);
  else y = sp ? scratch + d.loc_off : loc + d.loc_off;
  const int tid = threadIdx.x;
  const int32_t* col = S.scol + d.loc_off;
  const double* sc = S.sscale + d.loc_off;
  for (int q = tid; q < d.np; q += blockDim.x) y[q] = col[q] >= 0 ? sc[q] * rhs[col[q]] : 0.0;
  __syncthreads();
  const int r = tid % TS, g = tid / TS, ng = blockDim.x / TS;
  for (int I = 0; I < d.ntiles; ++I) {
    double acc = 0.0;
    for (int K = F[I] + g; K < I; K += ng) {
      const T* t = A + (off[I] + (K - F[I])) * TT;
      const double* yk = y + K * TS;
#pragma unroll 8
      for (int c = 0; c < TS; ++c) acc += (double)t[c * TS + r] * yk[c];
    }
    part[g][r] = acc;
    __syncthreads();
    if (tid < TS) {
      double s = y[I * TS + tid];
      for (int q = 0; q < ng; ++q) s -= part[q][tid];
      sv[tid] = s;
    }
    __syncthreads();
    if (tid < TS) {
      const T* inv = Di + (int64_t)I * TT;
      double s = 0.0;
#pragma unroll 8
      for (int c = 0; c < TS; ++c) s += (double)inv[c * TS + tid] * sv[c];
      y[I * TS + tid] = s;
    }
    __syncthreads();
  }
  for (int I = d.ntiles - 1; I >= 0; --I) {
    if (tid < TS) {
      const T* inv = Di + (int64_t)I * TT;
      double s = 0.0;
#pragma unroll 8
      for (int c = 0; c < TS; ++c) s += (double)inv[tid * TS + c] * y[I * TS + c];
      sv[tid] = s;
    }
    __syncthreads();
    if (tid < TS) y[I * TS + tid] = sv[tid];
    for (int K = F[I] + g; K < I; K += ng) {
      const T* t = A + (off[I] + (K - F[I])) * TT;
      double s = 0.0;
#pragma unroll 8
      for (int rr = 0; rr < TS; ++rr) s += (double)t[r * TS + rr] * sv[rr];
      y[K * TS + r] -= s;
    }
    __syncthreads();
  }
  for (int q = tid; q < d.np; q += blockDim.x)
    if (!sp) loc[d.loc_off + q] = sc[q] * y[q];
    else if (sp[q] >= 0) loc[sp[q]] = sc[q] * y[q];
}


// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
int local_solve_cap(bool f32) { return f32 ? SCAP_OF<float> : SCAP_OF<double>; }

void launch_stream_layout(hipStream_t st, int nsub, const DevPlan& P, const int32_t* F8,
                          const SubDesc* gsub, int64_t tiles, const SolveStream& S) {
  for (int dir = 0; dir < 2; ++dir) launch_fill_i32(st, 4 * tiles, -1, S.pos[dir]);
  k_stream_layout<<<nsub, 256, 0, st>>>(P.heavy(), P.tileF, P.tileOff, F8, gsub, S);
}

void launch_solve_cols(hipStream_t st, int nsub, const DevPlan& P, const DevPlan& Lay,
                       const double* scale, const SolveStream& S) {
  k_solve_cols<<<nsub, 256, 0, st>>>(P.heavy(), Lay.subs, P.omega, scale, Lay.sperm, S.scol, S.sscale);
}

template <typename T>
void launch_stream_pack(hipStream_t st, int nsub, const DevPlan& P, const T* fac, const T* dinv,
                        const SolveStream& S) {
  k_stream_pack<T><<<dim3(nsub, 16), 256, 0, st>>>(P.heavy(), P.tileF, P.tileOff, fac, dinv, S,
                                                    (T*)S.fwd, (T*)S.bwd, (T*)S.dpack);
}
template void launch_stream_pack<double>(hipStream_t, int, const DevPlan&, const double*, const double*,
                                         const SolveStream&);
template void launch_stream_pack<float>(hipStream_t, int, const DevPlan&, const float*, const float*,
                                        const SolveStream&);

template <typename T>
void launch_local_solve(hipStream_t st, int nsub, const DevPlan& P, const SolveStream& S, const T* fac,
                        const T* dinv, const double* r, double* loc) {
  const size_t lds = stream_lds_bytes(std::min(P.max_np, S.cap), sizeof(T));
  if (S.cap > 0)
    k_local_solve_stream<T><<<nsub, 64 * SOLVE_WAVES, lds, st>>>(P.heavy(), S, (const T*)S.fwd, (const T*)S.bwd,
                                                  (const T*)S.dpack, r, loc, P.sperm);
  else
    k_local_solve<T, true><<<nsub, 256, (size_t)std::min(P.max_np, SCAP) * sizeof(double), st>>>(
        P.subs, P.tileF, P.tileOff, fac, dinv, S, r, loc, P.sperm, P.yscratch, 0, SCAP);
  const int done = S.cap > 0 ? S.cap : SCAP;
  if (P.max_np > done)
    k_local_solve<T, false><<<nsub, 256, 0, st>>>(P.subs, P.tileF, P.tileOff, fac, dinv, S, r, loc, P.sperm,
                                                  P.yscratch, done, INT32_MAX);
}
template void launch_local_solve<double>(hipStream_t, int, const DevPlan&, const SolveStream&,
                                         const double*, const double*, const double*, double*);
template void launch_local_solve<float>(hipStream_t, int, const DevPlan&, const SolveStream&,
                                        const float*, const float*, const double*, double*);

hipError_t local_solve_configure() {
  hipError_t e = hipFuncSetAttribute((const void*)k_local_solve_stream<double>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)stream_lds_bytes(SCAP_OF<double>, sizeof(double)));
  if (e == hipSuccess)
    e = hipFuncSetAttribute((const void*)k_local_solve_stream<float>,
                            hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)stream_lds_bytes(SCAP_OF<float>, sizeof(float)));
  for (const void* k : {(const void*)k_local_solve<double, true>, (const void*)k_local_solve<float, true>})
    if (e == hipSuccess)
      e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, SCAP * (int)sizeof(double));
  return e;
}

}  // namespace lsq2l
