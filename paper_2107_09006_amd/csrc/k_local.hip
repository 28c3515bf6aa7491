// Subdomain kernels: local matrices, batched Cholesky, local solves.
//
//   C_ii  = A(:,Omega_i)^T A(:,Omega_i)            (Section 3.1)
//   Ct_GG = A(Xi_i,Omega_Gamma_i)^T A(Xi_i,Omega_Gamma_i)
//           (the only block in which the local SPSD splitting of
//            eq. spsd_normal_eq differs from C_ii: rows outside Xi_i have no
//            entry in Omega_Ii, so Ct_II = C_II and Ct_IG = C_IG)
//   C_ii  = L_i L_i^T                              (Algorithm 1, local Cholesky)
//   z_i   = C_ii^{-1} r_i                          (eq. one_level_schwarz)
//
// One workgroup owns one subdomain; subdomains of uneven size share a launch.
#include <algorithm>

#include "kernels.hpp"

namespace lsq2l {

// owner[e] = (part[c], locown[c]) of the column c of entry e
__global__ void k_entry_owner(int64_t nnz, const int32_t* __restrict__ colind, const int32_t* __restrict__ part,
                              const int32_t* __restrict__ locown, int2* __restrict__ owner) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= nnz) return;
  const int c = colind[e];
  owner[e] = int2{part[c], locown[c]};
}

// Lower triangle of C_ii (tile-envelope layout) and of Ct_GG (dense, ld nGp).
// Workgroup (i, y) takes the tile columns y, y + gridDim.y, ... of subdomain i,
// a wave CPW columns at a time: LPR lanes walk the entries of each row of A that
// holds the column, and every product is added in LDS at its row's place among
// the column's stored tiles.  All adds to an entry come from one wave: its steps follow
// one another, each over up to 64 / (CPW LPR) rows and LPR entries of each, and
// within a step the LDS adds lanes on one address in an order that is not
// documented (ascending lanes in every run observed, so results repeat).  The
// finished column is written once, zeros included, so the factor array needs
// no clearing.  Columns with more than NTL stored tiles take several passes over
// their rows.  owner[e] = (part, local position there) of the column of entry e,
// gathered once for all subdomains; without room for it (OWN false) the column's are
// looked up.
// With inv given, it also finds the envelope of C_ii in the global column order
// (see k_solve_inv): the wave of column a sees every column coupled to it, so
// the first coupled position of row inv[a] in that order is the minimum it
// meets, one atomicMin per column into F8 (one entry per eight rows).  With
// fac null that envelope is all it finds.
// With scl given (S = diag(C_ii)^{-1/2} per local position, which is
// 1 / ||A(:, c)||: C_ii holds whole columns of A), every product is scaled as it
// is added, so the result is S C_ii S and S Ct_GG S directly, with unit diagonal
// entries on the padding positions (the equilibration in one pass).
//
// What bounds it: the look-ups of the entries' positions and the factor array
// written once.  One thread per column, adding every product to its place in
// memory, took 14.7 ms (irregular, 1e6 columns, 4 GB of tiles, cleared before
// in 1.0) and 4.4 (batch of 3e6 columns, 3 GB); this takes 5.2 and 2.6.
constexpr int ASM_G = 1024;       // interface columns held in LDS
constexpr int ASM_MAP = 4096;     // tile rows with a direct slot table
template <int NTL, int CPW, int LPR, bool OWN>
__global__ void __launch_bounds__(256)
k_assemble(const SubDesc* __restrict__ subs, const int32_t* __restrict__ omega,
           const int2* __restrict__ owner, const int32_t* __restrict__ part,
           const int32_t* __restrict__ locown,
           const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colind,
           const double* __restrict__ vals, const int32_t* __restrict__ trowptr,
           const int32_t* __restrict__ trow, const double* __restrict__ tvals,
           const int32_t* __restrict__ tileF, const int64_t* __restrict__ tileOff,
           double* __restrict__ fac, double* __restrict__ ctg, const int32_t* __restrict__ inv,
           const SubDesc* __restrict__ gsub, int32_t* __restrict__ F8,
           const double* __restrict__ scl) {
  __shared__ __align__(16) double sAcc[4][CPW * NTL * TS];
  constexpr int SW = 64 / CPW;      // lanes of a column
  __shared__ int32_t sG[ASM_G], sList[NTL];
  __shared__ int64_t sBase[NTL];                // the stored tiles' places in A
  __shared__ __align__(16) double sScl[NTL * TS];             // S of their rows
  __shared__ uint8_t sMap[ASM_MAP];
  __shared__ int s_cnt, s_next;
  const SubDesc d = subs[blockIdx.x];
  const int i = d.id, tid = threadIdx.x, lane = tid % 64;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const double* sl = scl ? scl + d.loc_off : nullptr;
  const int32_t* iv = inv ? inv + d.loc_off : nullptr;
  const int32_t* om = omega + d.omega_off;
  const int32_t* G = om + d.nI;
  const int32_t* F = tileF + d.tile_base;
  const int64_t* off = tileOff + d.tile_base;
  double* A = fac ? fac + d.fac_off : nullptr;
  double* Ct = ctg ? ctg + d.g_off : nullptr;
  double* acc = sAcc[wave];
  const bool gl = d.nG <= ASM_G, map = d.ntiles <= ASM_MAP;
  if (gl)
    for (int q = tid; q < d.nG; q += 256) sG[q] = G[q];
  if (map)
    for (int q = tid; q < d.ntiles; q += 256) sMap[q] = 255;
  for (int q = lane; q < CPW * NTL * TS; q += 64) acc[q] = 0.0;
  __syncthreads();
  // local position of global column c owned by w, or -1
  auto position = [&](int c, int2 w) -> int {
    if (w.x == i) return w.y;
    int lo = 0, hi = d.nG;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if ((gl ? sG[mid] : G[mid]) < c) lo = mid + 1; else hi = mid;
    }
    return lo < d.nG && (gl ? sG[lo] : G[lo]) == c ? d.nIp + lo : -1;
  };
  for (int J = blockIdx.y; J < d.ntiles; J += gridDim.y) {
    int I0 = J;
    while (I0 < d.ntiles) {
      // the next (at most NTL) stored tiles of this tile column
      if (wave == 0) {
        int cnt = 0, at = I0;
        if (A) {
          while (at < d.ntiles && cnt < NTL) {
            const int I = at + lane;
            const bool fl = I < d.ntiles && F[I] <= J;
            const unsigned long long m = __ballot(fl);
            const int before = __popcll(m & ((1ull << lane) - 1ull));
            const bool take = fl && cnt + before < NTL;
            if (take) {
              sList[cnt + before] = I;
              if (map) sMap[I] = (uint8_t)(cnt + before);
            }
            const unsigned long long tk = __ballot(take);
            cnt += __popcll(tk);
            at += 64;
            if (tk != m) break;
          }
          wave_sync();
          if (cnt == NTL) at = sList[NTL - 1] + 1;   // a full list: resume after its last row
        } else {
          at = d.ntiles;
        }
        if (lane == 0) { s_cnt = cnt; s_next = at; }
      }
      __syncthreads();
      const int cnt = s_cnt, nextI = s_next;
      for (int q = tid; q < cnt; q += 256) sBase[q] = tile_pos(F, off, sList[q], J) * TT;
      if (sl)
        for (int q = tid; q < cnt * TS; q += 256) sScl[q] = sl[sList[q / TS] * TS + q % TS];
      __syncthreads();
      auto slot = [&](int I) -> int {
        if (map) return sMap[I] == 255 ? -1 : (int)sMap[I];
        int lo = 0, hi = cnt;
        while (lo < hi) {
          const int mid = (lo + hi) >> 1;
          if (sList[mid] < I) lo = mid + 1; else hi = mid;
        }
        return lo < cnt && sList[lo] == I ? lo : -1;
      };
      // column of group t and place u; lane t CPW + u holds the extent of its rows
      auto column = [&](int t, int u) { return J * TS + (4 * t + wave) * CPW + u; };
      int ext0 = 0, ext1 = 0;
      if (lane < TS / 4) {
        const int pos = column(lane / CPW, lane % CPW);
        const int at = pos < d.nI ? pos : pos >= d.nIp && pos < d.nIp + d.nG ? d.nI + pos - d.nIp : -1;
        if (at >= 0) {
          ext0 = trowptr[om[at]];
          ext1 = trowptr[om[at] + 1];
        }
      }
      const bool interior = J < d.ntI;                   // the whole tile column
      const int npass = !interior && Ct ? 2 : 1;         // C_ii, then Ct_GG (rows in Xi_i)
      for (int t = 0; t < TS / (4 * CPW); ++t) {
        const int u = lane / SW, pos = column(t, u);
        const int k0 = __shfl(ext0, t * CPW + u, 64), k1 = __shfl(ext1, t * CPW + u, 64);
        const bool real = k0 < k1;                       // every column of Omega_i has an entry
        double* mine = acc + u * (NTL * TS);
        const double sa = sl ? sl[pos] : 1.0;
        for (int pass = 0; pass < npass; ++pass) {
          const int qa = iv && real ? iv[pos] : 0;
          int fmin = qa;
          for (int k = k0 + lane % SW / LPR; k < k1; k += SW / LPR) {
            const int r = trow[k];
            const double va = tvals[k];
            const int e0 = rowptr[r], e1 = rowptr[r + 1];
            bool inxi = true;
            if (pass == 1) {
              inxi = false;
              for (int e = e0 + lane % LPR; e < e1; e += LPR) inxi |= (OWN ? owner[e].x : part[colind[e]]) == i;
              const unsigned long long m = __ballot(inxi);
              inxi = (m >> (lane & ~(LPR - 1))) & ((1ull << LPR) - 1ull);
            }
            if (!inxi) continue;
            for (int e = e0 + lane % LPR; e < e1; e += LPR) {
              const double v = vals[e];
              const int ce = colind[e];
              const int pc = position(ce, OWN ? owner[e] : int2{part[ce], locown[ce]});
              if (pc < 0) continue;
              if (iv) fmin = min(fmin, iv[pc]);
              if (!A || pc < pos) continue;
              const int sI = slot(pc / TS);
              if (sI < 0) continue;
              const int at = sI * TS + pc % TS;
              const double x = sl ? v * va * (sa * sScl[at]) : v * va;
              __builtin_amdgcn_ds_atomic_fadd_f64((__attribute__((address_space(3))) double*)(mine + at), x);
            }
          }
          if (iv && pass == 0 && I0 == J) {
#pragma unroll
            for (int o = SW / 2; o > 0; o >>= 1) fmin = min(fmin, __shfl_xor(fmin, o, 64));
            if (real && lane % SW == 0) atomicMin(&F8[4 * gsub[i].tile_base + qa / 8], fmin);
          }
          wave_sync();
#pragma unroll
          for (int w = 0; w < CPW; ++w) {
            const int pw = column(t, w);
            const bool rw = pw < d.nI || (pw >= d.nIp && pw < d.nIp + d.nG);
            double* from = acc + w * (NTL * TS);
            for (int s = lane / (TS / 2); s < cnt; s += 128 / TS) {
              const int rr = lane % (TS / 2) * 2, row = sList[s] * TS + rr;
              double2* at = reinterpret_cast<double2*>(from + s * TS + rr);
              double2 v = *at;
              *at = double2{0.0, 0.0};
              if (sl && !rw) {
                v.x = row == pw ? 1.0 : 0.0;
                v.y = row + 1 == pw ? 1.0 : 0.0;
              }
              if (pass == 0) *reinterpret_cast<double2*>(A + sBase[s] + (pw - J * TS) * TS + rr) = v;
              else if (row >= d.nIp)
                *reinterpret_cast<double2*>(Ct + (int64_t)(pw - d.nIp) * d.nGp + (row - d.nIp)) = v;
            }
          }
          wave_sync();
        }
      }
      __syncthreads();
      if (map && wave == 0)
        for (int q = lane; q < cnt; q += 64) sMap[sList[q]] = 255;
      __syncthreads();
      I0 = nextI;
    }
  }
}

// Symmetric diagonal equilibration S C S, S = diag(C)^{-1/2} (an exact
// congruence: C^{-1} = S (S C S)^{-1} S), applied to C_ii and to Ct_GG; the
// padding rows become identity rows.  scale[pos] = S_pos (0 on padding).
// k_equil_scale forms S per subdomain; k_equil_apply scales the stored tiles
// and Ct_GG, workgroup (i, y) taking tile rows y, y + gridDim.y, ...
__global__ void __launch_bounds__(256)
k_equil_scale(const SubDesc* __restrict__ subs, const int32_t* __restrict__ tileF,
              const int64_t* __restrict__ tileOff, const double* __restrict__ fac,
              double* __restrict__ scale) {
  const SubDesc d = subs[blockIdx.x];
  const int32_t* F = tileF + d.tile_base;
  const int64_t* off = tileOff + d.tile_base;
  const double* A = fac + d.fac_off;
  double* s = scale + d.loc_off;
  for (int pos = threadIdx.x; pos < d.np; pos += blockDim.x) {
    const bool real = pos < d.nI || (pos >= d.nIp && pos < d.nIp + d.nG);
    const double* diag = A + tile_pos(F, off, pos / TS, pos / TS) * TT + (pos % TS) * TS + pos % TS;
    s[pos] = real ? 1.0 / sqrt(*diag) : 0.0;   // diagonal > 0: every column of Omega_i has a stored entry
  }
}

__global__ void __launch_bounds__(256)
k_equil_apply(const SubDesc* __restrict__ subs, const int32_t* __restrict__ tileF,
              const int64_t* __restrict__ tileOff, double* __restrict__ fac,
              double* __restrict__ ctg, const double* __restrict__ scale) {
  const SubDesc d = subs[blockIdx.x];
  const int32_t* F = tileF + d.tile_base;
  const int64_t* off = tileOff + d.tile_base;
  double* A = fac + d.fac_off;
  const double* s = scale + d.loc_off;
  // pairs of entries (rows r, r + 1 of one column c) as 16-byte accesses
  typedef double d2 __attribute__((ext_vector_type(2)));
  for (int t = blockIdx.y; t < d.ntiles; t += gridDim.y) {
    const int nt = t - F[t] + 1;
    d2* row = reinterpret_cast<d2*>(A + off[t] * TT);
    for (int64_t e2 = threadIdx.x; e2 < (int64_t)nt * (TT / 2); e2 += blockDim.x) {
      const int64_t e = 2 * e2;
      const int J = F[t] + (int)(e / TT);
      const int rc = (int)(e % TT);
      const int r = t * TS + rc % TS, c = J * TS + rc / TS;
      const double sr0 = s[r], sr1 = s[r + 1], sc = s[c];
      d2 v = row[e2];
      v.x = (r == c && sr0 == 0.0) ? 1.0 : v.x * (sr0 * sc);
      v.y = (r + 1 == c && sr1 == 0.0) ? 1.0 : v.y * (sr1 * sc);
      row[e2] = v;
    }
  }
  double* Ct = ctg + d.g_off;
  for (int64_t e = (int64_t)blockIdx.y * blockDim.x + threadIdx.x; e < (int64_t)d.nGp * d.nGp;
       e += (int64_t)gridDim.y * blockDim.x) {
    const int r = (int)(e % d.nGp), c = (int)(e / d.nGp);
    Ct[e] *= s[d.nIp + r] * s[d.nIp + c];   // zero on padding
  }
}

constexpr int ROWCAP = 2048;
constexpr int CHOL_TMAX = 2048;   // tile rows whose envelope the factorization keeps in LDS

// Right-looking tile Cholesky of one envelope matrix per workgroup.  Step J
// starts with the diagonal tile J factored and inverted in LDS:
//   1. the panel tile (J + 1, J), if stored, L(I, J) = A(I, J) L(J, J)^{-T}, a
//      quarter on each of four waves;
//   2. the same quarters of A(J + 1, J + 1) - L(J + 1, J) L(J + 1, J)^T;
//   3. wave 0 factors that tile (for step J + 1) while the others store tile
//      J, list the rows of column J + 1, take the other panel tiles from a
//      counter and, once all are stored, the pairs of envelope rows
//      A(I, K) -= L(I, J) L(K, J)^T; wave 0 joins them when done.
// T is double or float (FP32 MFMA with FP32 accumulation).  With
// interior_only, the factor stops after the interior tile columns and the
// interface rows never update each other: the result holds L_I and L_GI only
// (what the coarse selection reads; the local solves then use factors of their
// own).
//
// What bounds it: on narrow envelopes the chain of the largest subdomain, per
// tile column the two quarter products, two barriers and the factorization of
// a tile by one wave; on wide ones the pairs (FP64 MFMA of one CU).  Batch of
// 64 banded problems (390 tile columns): 6.9 -> 4.2 ms; 512 irregular
// subdomains: 14.4 -> 9.9 ms, their FP32 solve factors 8.0 -> 4.1.  NT threads: see launch_chol.
template <typename T, int NT>
__global__ void __launch_bounds__(NT)
k_chol_local(const SubDesc* __restrict__ subs, const int32_t* __restrict__ tileF,
             const int64_t* __restrict__ tileOff, T* __restrict__ fac, T* __restrict__ dinv,
             int32_t* __restrict__ status, int interior_only) {
  using M = Mfma<T>;
  __shared__ T sW[TS * LDT], sP[TS * LDT], sL[2][TS * LDT], sInv[2][TS * LDT];
  __shared__ int32_t srows[2][ROWCAP];
  __shared__ uint16_t sF[CHOL_TMAX];
  __shared__ int32_t sO[CHOL_TMAX];
  __shared__ int s_count[2], s_ok[2], s_panel, s_done, s_pair;
  const SubDesc d = subs[blockIdx.x];
  const int32_t* F = tileF + d.tile_base;
  const int64_t* off = tileOff + d.tile_base;
  // the envelope (first tile column and offset of each tile row) in LDS, so
  // that finding a tile costs no global round trip
  const bool staged = d.ntiles <= CHOL_TMAX;
  if (staged)
    for (int I = threadIdx.x; I < d.ntiles; I += NT) {
      sF[I] = (uint16_t)F[I];
      sO[I] = (int32_t)off[I];
    }
  __syncthreads();
  auto first = [&](int I) -> int { return staged ? (int)sF[I] : F[I]; };
  auto tpos = [&](int I, int J) -> int64_t {
    return staged ? (int64_t)sO[I] + (J - (int)sF[I]) : tile_pos(F, off, I, J);
  };
  T* A = fac + d.fac_off;
  T* Di = dinv + d.dinv_off;
  constexpr int NW = NT / 64;
  const int tid = threadIdx.x, lane = tid % 64;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int li = lane % 16, lk = lane / 16;
  bool failed = false;
  // rows I > J whose envelope reaches column J, ascending, by one wave
  auto list_rows = [&](int J, int buf) {
    int cnt = 0;
    for (int base = J + 1; base < d.ntiles; base += 64) {
      const int I = base + lane;
      const bool fl = I < d.ntiles && first(I) <= J;
      const unsigned long long mask = __ballot(fl);
      const int before = __popcll(mask & ((1ull << lane) - 1ull));
      if (fl && cnt + before < ROWCAP) srows[buf][cnt + before] = I;
      cnt += __popcll(mask);
    }
    if (lane == 0) s_count[buf] = cnt;
  };
  auto next_item = [&](int* counter) {
    int it = 0;
    if (lane == 0) it = atomicAdd(counter, 1);
    return __builtin_amdgcn_readfirstlane(it);
  };
  // tile columns to factor, and the first row of the block whose mutual
  // updates are skipped
  const int ncol = interior_only ? d.ntI : d.ntiles;
  const int skip_from = interior_only ? d.ntI : d.ntiles;
  if (wave == 0 && ncol > 0) {
    const T* A00 = A + tpos(0, 0) * TT;
    for (int e = lane; e < TT; e += 64) sW[(e / TS) * LDT + e % TS] = A00[e];
    wave_sync();
    const bool okw = tile_potrf_inv(sW, sL[0], sInv[0], lane);
    if (lane == 0) s_ok[0] = okw;
  } else if (wave == NW - 1) {
    list_rows(0, 0);
  }
  __syncthreads();
  for (int J = 0; J < ncol; ++J) {
    const int cur = J & 1;
    const int32_t* rows = srows[cur];
    const int nr = s_count[cur];
    if (!s_ok[cur]) failed = true;
    if (nr > ROWCAP) { failed = true; break; }
    const bool next = J + 1 < ncol;
    const bool coupled = nr > 0 && rows[0] == J + 1;
    // quarter (bi, bj) of a transposed tile: columns 16 bi .., rows 16 bj ..
    const int bi = wave / 2, bj = wave % 2;
    const bool quarter = next && wave < 4 && !(bi == 1 && bj == 0);   // lower part only
    typename M::acc_t q;
    const T* Ann = A + (next ? tpos(J + 1, J + 1) : 0) * TT;
    if (quarter)
#pragma unroll
      for (int v = 0; v < 4; ++v) q[v] = Ann[(16 * bi + M::acc_row(lane, v)) * TS + 16 * bj + li];
    if (coupled && wave < 4) {
      T* Pn = A + tpos(J + 1, J) * TT;
      T b[8];
#pragma unroll
      for (int s = 0; s < 8; ++s) b[s] = Pn[(4 * s + lk) * TS + 16 * bj + li];
      typename M::acc_t acc = M::zero();
#pragma unroll
      for (int s = 0; s < 8; ++s) acc = M::mma(sInv[cur][(4 * s + lk) * LDT + 16 * bi + li], b[s], acc);
#pragma unroll
      for (int v = 0; v < 4; ++v) sP[(16 * bi + M::acc_row(lane, v)) * LDT + 16 * bj + li] = acc[v];
    }
    if (tid == 0) {
      s_panel = s_done = coupled ? 1 : 0;
      s_pair = coupled && next ? 1 : 0;
    }
    __syncthreads();                     // the quarters read all of A(J + 1, J) before it is overwritten
    if (coupled) {
      T* Pn = A + tpos(J + 1, J) * TT;
      for (int e = tid; e < TT; e += NT) Pn[e] = sP[(e / TS) * LDT + e % TS];
      if (quarter) {
#pragma unroll
        for (int s = 0; s < 8; ++s)
          q = M::mma(-sP[(4 * s + lk) * LDT + 16 * bi + li], sP[(4 * s + lk) * LDT + 16 * bj + li], q);
      }
    }
    if (quarter)
#pragma unroll
      for (int v = 0; v < 4; ++v) sW[(16 * bi + M::acc_row(lane, v)) * LDT + 16 * bj + li] = q[v];
    __syncthreads();
    if (wave == 0 && next) {
      const bool okw = tile_potrf_inv(sW, sL[cur ^ 1], sInv[cur ^ 1], lane);
      if (lane == 0) s_ok[cur ^ 1] = okw;
    } else {
      if (wave == NW - 1 && next) list_rows(J + 1, cur ^ 1);
      T* Ajj = A + tpos(J, J) * TT;
      const int t0 = next ? tid - 64 : tid, nt = next ? NT - 64 : NT;
      for (int e = t0; e < TT; e += nt) {
        Ajj[e] = sL[cur][(e / TS) * LDT + e % TS];
        Di[(int64_t)J * TT + e] = sInv[cur][(e / TS) * LDT + e % TS];
      }
    }
    for (int it = next_item(&s_panel); it < nr; it = next_item(&s_panel)) {
      T* Aij = A + tpos(rows[it], J) * TT;
      typename M::acc_t acc[4];
      tile_acc_zero<T>(acc);
      tile_mma_nt<T, false>(acc, sInv[cur], LDT, Aij, TS, lane);
      tile_accT_store<T>(acc, Aij, TS, lane);
      wg_fence();
      if (lane == 0) atomicAdd(&s_done, 1);
    }
    // every panel tile is taken by now, and the waves that took them do not wait
    while (*(volatile int*)&s_done < nr) __builtin_amdgcn_s_sleep(1);
    wg_fence();
    const int npairs = nr * (nr + 1) / 2;
    for (int it = next_item(&s_pair); it < npairs; it = next_item(&s_pair)) {
      int a = (int)((sqrt(8.0 * it + 1.0) - 1.0) / 2.0);
      while (a * (a + 1) / 2 > it) --a;
      while ((a + 1) * (a + 2) / 2 <= it) ++a;
      const int b = it - a * (a + 1) / 2;
      const int Ia = rows[a], Ib = rows[b];
      if (Ib >= skip_from) continue;     // both rows at or past skip_from (rows ascend)
      const T* La = A + tpos(Ia, J) * TT;
      const T* Lb = A + tpos(Ib, J) * TT;
      T* Cab = A + tpos(Ia, Ib) * TT;
      typename M::acc_t acc[4];
      tile_accT_load<T>(acc, Cab, TS, lane);
      tile_mma_nt<T, true>(acc, Lb, TS, La, TS, lane);
      tile_accT_store<T>(acc, Cab, TS, lane);
    }
    __syncthreads();
  }
  if (failed && tid == 0) atomicCAS(status, 0, d.id + 1);
}

// ---------------------------------------------------------------------------
// The factor used by the per-iteration local solves.  C_ii^{-1} r does not
// depend on the order of Omega_i, and the order [Omega_Ii, Omega_Gamma_i]
// that the coarse selection needs (T = L_GI L_GI^T) makes the interface rows
// of L dense across the interior.  The solve factor therefore orders
// Omega_i by global column (the order of the columns of A) where that stores
// fewer tiles: position q of that order is the q-th smallest column of
// Omega_i.  Its envelope comes from the assembled C_ii itself (the first
// nonzero of each row after the permutation), which the factorization
// cannot leave; its values are gathered from the assembled, equilibrated
// C_ii before that is factored in place.
// ---------------------------------------------------------------------------

// inv[loc_off + pos] = position of the column at [I, Gamma] position pos in
// the global-column order of Omega_i (-1 on padding): the column's rank
// among the interior columns plus its rank among the interface columns
__global__ void __launch_bounds__(256)
k_solve_inv(const SubDesc* __restrict__ subs, const int32_t* __restrict__ omega,
            int32_t* __restrict__ inv) {
  const SubDesc d = subs[blockIdx.x];
  const int32_t* om = omega + d.omega_off;
  const int32_t* G = om + d.nI;
  auto rank = [](const int32_t* v, int n, int32_t c) {   // entries of v below c
    int lo = 0, hi = n;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (v[mid] < c) lo = mid + 1; else hi = mid;
    }
    return lo;
  };
  for (int pos = threadIdx.x; pos < d.np; pos += blockDim.x) {
    int q = -1;
    if (pos < d.nI) q = pos + rank(G, d.nG, om[pos]);
    else if (pos >= d.nIp && pos < d.nIp + d.nG) q = (pos - d.nIp) + rank(om, d.nI, G[pos - d.nIp]);
    inv[d.loc_off + pos] = q;
  }
}

// F8[4 tile_base + g] = 8 g for every group g of eight rows of the global-order layout
__global__ void __launch_bounds__(256)
k_solve_env_init(const SubDesc* __restrict__ gsub, int32_t* __restrict__ F8) {
  const SubDesc g = gsub[blockIdx.x];
  for (int t = threadIdx.x; t < 4 * g.ntiles; t += blockDim.x) F8[4 * g.tile_base + t] = 8 * t;
}

// first tile column of tile row t from the envelope of its four row groups
__device__ inline int first_tile(const int32_t* f8, int t) {
  return min(min(f8[4 * t], f8[4 * t + 1]), min(f8[4 * t + 2], f8[4 * t + 3])) / TS;
}

// tiles[i] = tiles of the envelope of subdomain i's global-order layout
__global__ void __launch_bounds__(256)
k_layout_count(const SubDesc* __restrict__ gsub, const int32_t* __restrict__ F8, int32_t* __restrict__ tiles) {
  __shared__ int sh[4];
  const SubDesc g = gsub[blockIdx.x];
  const int32_t* f8 = F8 + 4 * g.tile_base;
  int v = 0, total = 0;
  for (int t = threadIdx.x; t < g.ntiles; t += 256) v += t - first_tile(f8, t) + 1;
  (void)block_excl_scan_256(v, sh, &total);
  if (threadIdx.x == 0) tiles[blockIdx.x] = total;
}

// envelope tables of the chosen layouts: from F8 where ssub.spare is set, else
// those of the [I, Gamma] layout; offsets are the running tile counts
__global__ void __launch_bounds__(256)
k_layout_fill(const SubDesc* __restrict__ subs, const int32_t* __restrict__ tileF,
              const SubDesc* __restrict__ ssub, const SubDesc* __restrict__ gsub,
              const int32_t* __restrict__ F8, int32_t* __restrict__ stileF, int64_t* __restrict__ stileOff) {
  __shared__ int sh[4];
  const SubDesc d = subs[blockIdx.x];
  const SubDesc s = ssub[d.id];
  const int32_t* f8 = F8 + 4 * gsub[d.id].tile_base;
  int run = 0;
  for (int t0 = 0; t0 < s.ntiles; t0 += 256) {
    const int t = t0 + threadIdx.x;
    int f = 0, n = 0, total = 0;
    if (t < s.ntiles) {
      f = s.spare ? first_tile(f8, t) : tileF[d.tile_base + t];
      n = t - f + 1;
    }
    const int before = run + block_excl_scan_256(n, sh, &total);
    if (t < s.ntiles) {
      stileF[s.tile_base + t] = f;
      stileOff[s.tile_base + t] = before;
    }
    run += total;
  }
}

// sperm[loc_off + q] = loc index of the entry the solve layout holds at
// position q (-1: padding): the global-column order where ssub.spare is set,
// the [I, Gamma] layout itself otherwise.  sperm is -1 on entry.
__global__ void __launch_bounds__(256)
k_solve_perm(const SubDesc* __restrict__ subs, const SubDesc* __restrict__ ssub,
             const int32_t* __restrict__ inv, int32_t* __restrict__ sperm) {
  const SubDesc d = subs[blockIdx.x];
  const SubDesc s = ssub[d.id];
  for (int pos = threadIdx.x; pos < d.np; pos += blockDim.x) {
    if (s.spare) {
      const int q = inv[d.loc_off + pos];
      if (q >= 0) sperm[s.loc_off + q] = (int32_t)(d.loc_off + pos);
    } else {
      sperm[s.loc_off + pos] = (int32_t)(d.loc_off + pos);
    }
  }
}

constexpr int GATHER_TMAX = 2048;

// The solve layout's matrix (tile envelope, double) from the assembled and
// equilibrated [I, Gamma] C_ii: entry (q_r, q_c) is C_ii(p_r, p_c) with
// p = sperm - loc_off, zero outside the [I, Gamma] envelope, and the
// identity on padding.  Workgroup (i, y) writes tile rows y, y + gridDim.y, ...
__global__ void __launch_bounds__(256)
k_gather_solve(const SubDesc* __restrict__ subs, const SubDesc* __restrict__ ssub,
               const int32_t* __restrict__ tileF, const int64_t* __restrict__ tileOff,
               const double* __restrict__ fac, const int32_t* __restrict__ stileF,
               const int64_t* __restrict__ stileOff, const int32_t* __restrict__ sperm,
               double* __restrict__ out) {
  __shared__ int32_t lF[GATHER_TMAX], lO[GATHER_TMAX];
  const SubDesc d = subs[blockIdx.x];
  const SubDesc s = ssub[d.id];
  const int32_t* F = tileF + d.tile_base;
  const int64_t* off = tileOff + d.tile_base;
  const double* A = fac + d.fac_off;
  const int32_t* Fs = stileF + s.tile_base;
  const int64_t* offs = stileOff + s.tile_base;
  const int32_t* sp = sperm + s.loc_off;
  double* O = out + s.fac_off;
  // the [I, Gamma] envelope table in LDS (looked up for every entry)
  const bool staged = d.ntiles <= GATHER_TMAX;
  if (staged)
    for (int I = threadIdx.x; I < d.ntiles; I += blockDim.x) {
      lF[I] = F[I];
      lO[I] = (int32_t)off[I];
    }
  __syncthreads();
  for (int I = blockIdx.y; I < s.ntiles; I += gridDim.y) {
    const int nk = I - Fs[I] + 1;
    double* row = O + offs[I] * TT;
    for (int e = threadIdx.x; e < nk * TT; e += blockDim.x) {
      const int J = Fs[I] + e / TT, rc = e % TT;
      const int qr = I * TS + rc % TS, qc = J * TS + rc / TS;
      const int pr = sp[qr], pc = sp[qc];
      double v;
      if (pr < 0 || pc < 0) {
        v = (qr == qc) ? 1.0 : 0.0;
      } else {
        const int hi = (int)(max(pr, pc) - d.loc_off), lo = (int)(min(pr, pc) - d.loc_off);
        const int th = hi / TS, tl = lo / TS;
        const int fh = staged ? lF[th] : F[th];
        const int64_t t = staged ? (int64_t)lO[th] + (tl - fh) : tile_pos(F, off, th, tl);
        v = tl >= fh ? A[t * TT + (lo % TS) * TS + hi % TS] : 0.0;
      }
      row[e] = v;
    }
  }
}

__global__ void k_to_float(int64_t n, const double* __restrict__ src, float* __restrict__ dst) {
  int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) dst[k] = (float)src[k];
}

// z_j = sum over the subdomains holding column j of loc_pos (fixed order), plus the coarse prolongation X_i d_i on the interior of its owner.
// Without loc only the prolongation is formed, without dcoarse only the sum.
// With `restricted`, column j takes only the value of its own subdomain's
// interior (R_i^T D_i of eq. RAS: D_i is zero on Omega_Gamma_i).
template <typename TX>
__global__ void k_scatter_local(int32_t n, const int32_t* __restrict__ own_ptr,
                                const int32_t* __restrict__ own_pos, const double* __restrict__ loc, const int32_t* __restrict__ part,
                                const int32_t* __restrict__ locown, const SubDesc* __restrict__ subs,
                                const TX* __restrict__ X, const double* __restrict__ dcoarse,
                                double* __restrict__ z, int restricted) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  double s = 0.0;
  if (loc != nullptr) {
    if (restricted) {
      const int64_t pos = subs[part[j]].loc_off + locown[j];
      s = loc[pos];
    } else {
      for (int q = own_ptr[j]; q < own_ptr[j + 1]; ++q) {
        s += loc[own_pos[q]];
      }
    }
  }
  if (dcoarse != nullptr) {
    const SubDesc d = subs[part[j]];
    const int a = locown[j];
    const TX* xr = X + d.x_off + a;
    const double* dc = dcoarse + d.cg_off;
    // eight independent loads in flight per thread
    double c8[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    int k = 0;
    for (; k + 8 <= d.p; k += 8)
#pragma unroll
      for (int i = 0; i < 8; ++i) c8[i] += (double)xr[(int64_t)(k + i) * d.nIp] * dc[k + i];
    for (int i = 0; k < d.p; ++k, ++i) c8[i] += (double)xr[(int64_t)k * d.nIp] * dc[k];
    s += ((c8[0] + c8[1]) + (c8[2] + c8[3])) + ((c8[4] + c8[5]) + (c8[6] + c8[7]));
  }
  z[j] = s;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
void launch_entry_owner(hipStream_t st, const DevPlan& P, const DevMatrix& M, int2* owner) {
  if (M.nnz == 0) return;
  k_entry_owner<<<(unsigned)((M.nnz + 255) / 256), 256, 0, st>>>(M.nnz, M.colind, P.part, P.locown, owner);
}

// Rows of up to four entries on average (a grid's edges have two, the banded
// rows four) fill four lanes each, and two columns at a time hide the loads'
// latency (batch of 3e6 banded columns 2.6 ms, grid of 1e6 1.0; one column and
// eight lanes 3.3 and 1.2).  Longer rows take eight lanes, one column and 16
// slots, for their wider envelopes (irregular, 1e6 columns, rows of 1 to 40:
// 5.2 ms; two columns and four lanes 7.0).
void launch_assemble(hipStream_t st, int nsub, const DevPlan& P, const DevMatrix& M, const int2* owner,
                     double* fac, double* ctg, const int32_t* inv, const SubDesc* gsub, int32_t* F8,
                     const double* scale) {
  // workgroups per subdomain: two tile columns each in a subdomain of 1,024
  // positions, at most 32
  const int ny = std::max(1, std::min(32, P.max_np / (2 * TS)));
  const bool few = M.nnz <= 4 * (int64_t)M.m;
  auto* kernel = owner ? (few ? k_assemble<8, 2, 4, true> : k_assemble<16, 1, 8, true>)
                       : (few ? k_assemble<8, 2, 4, false> : k_assemble<16, 1, 8, false>);
  kernel<<<dim3(nsub, ny), 256, 0, st>>>(P.heavy(), P.omega, owner, P.part, P.locown, M.rowptr, M.colind, M.vals, M.trowptr,
                                         M.trow, M.tvals, P.tileF, P.tileOff, fac, ctg, inv, gsub, F8, scale);
}

void launch_equilibrate(hipStream_t st, int nsub, const DevPlan& P, double* fac, double* ctg,
                        double* scale) {
  k_equil_scale<<<nsub, 256, 0, st>>>(P.heavy(), P.tileF, P.tileOff, fac, scale);
  k_equil_apply<<<dim3(nsub, 32), 256, 0, st>>>(P.heavy(), P.tileF, P.tileOff, fac, ctg, scale);
}

// Eight waves per subdomain where a tile column has many rows (the pairs of
// rows are shared out among them), four on narrow envelopes, where the chain of
// the diagonal tiles bounds the factorization and a workgroup that fits beside
// the selection's kernels is worth more.  512 irregular subdomains (10 tiles
// per row) 9.9 ms with eight waves, 11.9 with four; 1000 x 1000 grid, factors of
// the selection (7 tiles per row) 2.2 and 2.4, solve factors (3 per row) with
// the selection beside them 17.1 and 15.7.
template <typename T>
static void launch_chol(hipStream_t st, int nsub, const DevPlan& P, int64_t tiles, int64_t rows, T* fac,
                        T* dinv, int32_t* status, int interior_only) {
  if (tiles >= 6 * rows)
    k_chol_local<T, 512><<<nsub, 512, 0, st>>>(P.heavy(), P.tileF, P.tileOff, fac, dinv, status,
                                               interior_only);
  else
    k_chol_local<T, 256><<<nsub, 256, 0, st>>>(P.heavy(), P.tileF, P.tileOff, fac, dinv, status,
                                               interior_only);
}

void launch_chol_local(hipStream_t st, int nsub, const DevPlan& P, int64_t tiles, int64_t rows, double* fac,
                       double* dinv, int32_t* status, bool interior_only) {
  launch_chol<double>(st, nsub, P, tiles, rows, fac, dinv, status, interior_only ? 1 : 0);
}

void launch_solve_inv(hipStream_t st, int nsub, const DevPlan& P, int32_t* inv) {
  k_solve_inv<<<nsub, 256, 0, st>>>(P.heavy(), P.omega, inv);
}

void launch_layout_count(hipStream_t st, int nsub, const SubDesc* gsub, const int32_t* F8, int32_t* tiles) {
  k_layout_count<<<nsub, 256, 0, st>>>(gsub, F8, tiles);
}

void launch_layout_fill(hipStream_t st, int nsub, const DevPlan& P, const SubDesc* ssub,
                        const SubDesc* gsub, const int32_t* F8, int32_t* tileF, int64_t* tileOff) {
  k_layout_fill<<<nsub, 256, 0, st>>>(P.heavy(), P.tileF, ssub, gsub, F8, tileF, tileOff);
}

void launch_solve_env_init(hipStream_t st, int nsub, const SubDesc* gsub, int32_t* F8) {
  k_solve_env_init<<<nsub, 256, 0, st>>>(gsub, F8);
}

void launch_solve_perm(hipStream_t st, int nsub, const DevPlan& P, const SubDesc* ssub,
                       const int32_t* inv, int32_t* sperm) {
  k_solve_perm<<<nsub, 256, 0, st>>>(P.heavy(), ssub, inv, sperm);
}

void launch_gather_solve(hipStream_t st, int nsub, const DevPlan& P, const DevPlan& Ps,
                         const double* fac, double* out) {
  k_gather_solve<<<dim3(nsub, 16), 256, 0, st>>>(P.heavy(), Ps.subs, P.tileF, P.tileOff, fac,
                                                  Ps.tileF, Ps.tileOff, Ps.sperm, out);
}

void launch_chol_local_f32(hipStream_t st, int nsub, const DevPlan& P, int64_t tiles, int64_t rows,
                           float* fac, float* dinv, int32_t* status) {
  launch_chol<float>(st, nsub, P, tiles, rows, fac, dinv, status, 0);
}

void launch_to_float(hipStream_t st, int64_t n, const double* src, float* dst) {
  if (n == 0) return;
  k_to_float<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(n, src, dst);
}

void launch_scatter_local(hipStream_t st, int32_t n, const DevPlan& P, const double* loc,
                          const double* X, const double* dcoarse, double* z, bool restricted) {
  if (n == 0) return;
  k_scatter_local<double><<<(n + 255) / 256, 256, 0, st>>>(n, P.own_ptr, P.own_pos, loc,
                                                           P.part, P.locown, P.subs, X, dcoarse, z,
                                                           restricted ? 1 : 0);
}

void launch_scatter_local(hipStream_t st, int32_t n, const DevPlan& P, const double* loc,
                          const float* X, const double* dcoarse, double* z, bool restricted) {
  if (n == 0) return;
  k_scatter_local<float><<<(n + 255) / 256, 256, 0, st>>>(n, P.own_ptr, P.own_pos, loc,
                                                          P.part, P.locown, P.subs, X, dcoarse, z,
                                                          restricted ? 1 : 0);
}

// ||C(Omega_Ii, :)||_F^2 from the lower triangle of the assembled C_ii: the
// rows of C owned by subdomain i are its interior rows, and every column
// they couple to lies in Omega_i.  Entries (r, c), r >= c, count twice when
// both are interior (the upper mirror), once on the diagonal and once in the
// (Gamma, I) block; the (Gamma, Gamma) block belongs to other subdomains.
// One workgroup per subdomain, the sum in a fixed order.
__global__ void __launch_bounds__(256)
k_frob_interior(const SubDesc* __restrict__ subs, const int32_t* __restrict__ tileF,
                const int64_t* __restrict__ tileOff, const double* __restrict__ fac,
                double* __restrict__ out) {
  __shared__ double sh[4];
  const SubDesc d = subs[blockIdx.x];
  const int32_t* F = tileF + d.tile_base;
  const int64_t* off = tileOff + d.tile_base;
  const double* A = fac + d.fac_off;
  double acc = 0.0;
  for (int t = 0; t < d.ntiles; ++t) {
    const int nt = t - F[t] + 1;
    const double* row = A + off[t] * TT;
    for (int64_t e = threadIdx.x; e < (int64_t)nt * TT; e += blockDim.x) {
      const int J = F[t] + (int)(e / TT);
      const int rc = (int)(e % TT);
      const int r = t * TS + rc % TS, c = J * TS + rc / TS;
      if (r < c || c >= d.nI) continue;      // upper part, or a column outside the interior
      const double v = row[e];
      const double wgt = (r < d.nI) ? (r == c ? 1.0 : 2.0) : 1.0;
      acc += wgt * v * v;
    }
  }
  acc = wave_allsum(acc);
  if (threadIdx.x % 64 == 0) sh[threadIdx.x / 64] = acc;
  __syncthreads();
  if (threadIdx.x == 0) out[blockIdx.x] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// C_ii += s I on the positions of real columns (the padding keeps its zero
// diagonal until the equilibration turns it into identity rows)
__global__ void __launch_bounds__(256)
k_add_diag(const SubDesc* __restrict__ subs, const int32_t* __restrict__ tileF,
           const int64_t* __restrict__ tileOff, double s, double* __restrict__ fac) {
  const SubDesc d = subs[blockIdx.x];
  const int32_t* F = tileF + d.tile_base;
  const int64_t* off = tileOff + d.tile_base;
  double* A = fac + d.fac_off;
  for (int pos = threadIdx.x; pos < d.np; pos += blockDim.x) {
    const bool real = pos < d.nI || (pos >= d.nIp && pos < d.nIp + d.nG);
    if (real) A[tile_pos(F, off, pos / TS, pos / TS) * TT + (pos % TS) * TS + pos % TS] += s;
  }
}

void launch_frob_interior(hipStream_t st, int nsub, const DevPlan& P, const double* fac,
                          double* out) {
  k_frob_interior<<<nsub, 256, 0, st>>>(P.subs, P.tileF, P.tileOff, fac, out);
}

void launch_add_diag(hipStream_t st, int nsub, const DevPlan& P, double s, double* fac) {
  k_add_diag<<<nsub, 256, 0, st>>>(P.subs, P.tileF, P.tileOff, s, fac);
}

}  // namespace lsq2l
