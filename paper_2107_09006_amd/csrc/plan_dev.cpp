#include "plan_dev.hpp"

#include <cstring>
#include <string>

namespace lsq2l {
namespace {

// Stable sorts of CSR patterns by column (transposes) and scans on one
// stream, through work space that is shared by all of them and grows.
struct Sorter {
  hipStream_t st;
  Scratch& tmp;
  char* w = nullptr;
  size_t have = 0;
  lsq2l_status need(size_t bytes) {
    if (bytes <= have) return LSQ2L_OK;
    TRY(tmp.alloc(&w, (int64_t)bytes));
    have = bytes;
    return LSQ2L_OK;
  }
  lsq2l_status sort(int32_t m, int32_t n, int64_t nnz, const int32_t* rowptr, const int32_t* colind,
                    int32_t* tptr, int32_t* trow, int32_t* tperm) {
    const size_t b = transpose_temp_bytes(nnz, n);
    TRY(need(b));
    LSQ2L_HIP_TRY(launch_transpose(st, m, n, nnz, rowptr, colind, nullptr, tptr, trow, nullptr, tperm, w, b));
    return LSQ2L_OK;
  }
  lsq2l_status scan(int64_t n, int32_t* v) {
    TRY(need((size_t)scan_work_len(n) * sizeof(int32_t)));
    launch_exclusive_scan(st, n, v, (int32_t*)w);
    return LSQ2L_OK;
  }
  // keys (ascending inside the segments of ptr) without repeats: out and optr
  lsq2l_status distinct(int32_t nseg, int64_t len, const int32_t* ptr, const int32_t* key, int32_t* first,
                        int32_t* out, int32_t* optr) {
    launch_seg_first(st, nseg, len, ptr, key, first);
    TRY(scan(len + 1, first));
    launch_seg_pack(st, nseg, len, ptr, key, first, out, optr);
    return LSQ2L_OK;
  }
};

}  // namespace

lsq2l_status plan_build_device(lsq2l_ctx* c, int32_t nparts, const std::vector<int32_t>& seg_of_part,
                               int2* owner, Scratch& keep, DevicePlan& out) {
  const hipStream_t st = c->st;
  const DevMatrix& M = c->M;
  const int32_t m = M.m, n = M.n;
  const int64_t nnz = M.nnz;
  HostPlan& H = c->H;
  Scratch tmp(st);
  Sorter S{st, tmp};
  PinnedArray<int32_t> back;               // what the host reads of the device's counts
  TRY(back.alloc(3 * ((int64_t)nparts + 1) + 16));
  auto read = [&](const void* src, size_t bytes, size_t at) -> hipError_t {
    return hipMemcpyAsync((char*)back.p + at, src, bytes, hipMemcpyDeviceToHost, st);
  };
  // rows and columns are walked by a few lanes: no long ones
  unsigned long long* size = nullptr;      // two of k_plan_stat, three of k_plan_size
  unsigned long long stat[2], sz[3];
  TRY(tmp.alloc(&size, 5));
  LSQ2L_HIP_TRY(hipMemsetAsync(size, 0, 5 * sizeof(unsigned long long), st));
  launch_plan_stat(st, M, ROW_ORDER_JUMP, size);
  LSQ2L_HIP_TRY(read(size, sizeof(stat), 0));
  LSQ2L_HIP_TRY(hipStreamSynchronize(st));
  std::memcpy(stat, back.p, sizeof(stat));
  if (stat[0] > DEVICE_PLAN_LONGEST) return LSQ2L_OK;
  out.far_descents = (int64_t)stat[1];
  // columns of every part, ascending, and each column's position in its part
  int32_t *iota = nullptr, *pptr = nullptr, *pcols = nullptr, *unused = nullptr;
  const int64_t longest = std::max(m, n);
  TRY(tmp.alloc(&iota, longest + 1));
  TRY(tmp.alloc(&pptr, (int64_t)nparts + 1));
  TRY(tmp.alloc(&pcols, n));
  TRY(tmp.alloc(&unused, std::max<int64_t>(nnz, longest)));
  launch_iota(st, longest + 1, iota);
  TRY(S.sort(n, nparts, n, iota, c->P.part, pptr, pcols, unused));
  TRY(c->dalloc(&c->P.locown, n));
  launch_locown(st, n, pcols, c->P.part, pptr, c->P.locown);
  launch_entry_owner(st, c->P, M, owner);
  // Xi_i: the parts along every row, sorted by part, without repeats
  int32_t *rptr = nullptr, *rpart = nullptr, *aptr = nullptr, *arow = nullptr, *first = nullptr;
  int32_t *xi = nullptr, *xoff = nullptr;
  TRY(tmp.alloc(&rptr, (int64_t)m + 1));
  TRY(tmp.alloc(&aptr, (int64_t)nparts + 1));
  TRY(tmp.alloc(&xoff, (int64_t)nparts + 1));
  launch_row_runs(st, m, M.rowptr, owner, rptr, nullptr);
  TRY(S.scan((int64_t)m + 1, rptr));
  LSQ2L_HIP_TRY(read(rptr + m, sizeof(int32_t), 0));
  LSQ2L_HIP_TRY(hipStreamSynchronize(st));
  const int64_t nruns = back.p[0];
  TRY(tmp.alloc(&rpart, nruns));
  TRY(tmp.alloc(&arow, nruns));
  TRY(tmp.alloc(&first, nruns + 1));
  launch_row_runs(st, m, M.rowptr, owner, rptr, rpart);
  TRY(S.sort(m, nparts, nruns, rptr, rpart, aptr, arow, unused));
  xi = rpart;                              // read no more
  TRY(S.distinct(nparts, nruns, aptr, arow, first, xi, xoff));
  LSQ2L_HIP_TRY(read(xoff, ((size_t)nparts + 1) * sizeof(int32_t), 0));
  LSQ2L_HIP_TRY(hipStreamSynchronize(st));
  const int64_t nx = back.p[nparts];
  TRY(c->dalloc(&c->P.xi, nx));
  LSQ2L_HIP_TRY(hipMemcpyAsync(c->P.xi, xi, nx * sizeof(int32_t), hipMemcpyDeviceToDevice, st));
  xi = c->P.xi;
  // the parts of every row, ascending, with the row's place in their Xi
  int32_t *qptr = nullptr, *qpart = nullptr, *qperm = nullptr, *cptr = nullptr;
  TRY(tmp.alloc(&qptr, (int64_t)m + 1));
  TRY(tmp.alloc(&qpart, nx));
  TRY(tmp.alloc(&qperm, nx));
  TRY(tmp.alloc(&cptr, (int64_t)n + 1));
  TRY(S.sort(nparts, m, nx, xoff, xi, qptr, qpart, qperm));
  launch_plan_size(st, m, M.rowptr, qptr, size + 2);
  LSQ2L_HIP_TRY(read(size + 2, sizeof(sz), 0));
  LSQ2L_HIP_TRY(hipStreamSynchronize(st));
  std::memcpy(sz, back.p, sizeof(sz));
  const unsigned long long most = std::min<unsigned long long>(8ull * nnz, 1ull << 30);
  if (sz[0] > most || sz[1] > most || sz[2] > DEVICE_PLAN_LONGEST) return LSQ2L_OK;
  const int64_t npairs = (int64_t)sz[1];
  // Omega_Gamma_i: the other parts met along every column, sorted by part
  launch_col_parts(st, n, M.trowptr, M.trow, qptr, qpart, c->P.part, cptr, nullptr);
  TRY(S.scan((int64_t)n + 1, cptr));
  int32_t *cpart = nullptr, *bptr = nullptr, *bcol = nullptr, *bperm = nullptr, *gfirst = nullptr;
  int32_t *gamma = nullptr, *goff = nullptr;
  const int64_t ncand = (int64_t)sz[0];    // the scan's total: L (k - 1) over the rows
  TRY(tmp.alloc(&cpart, ncand));
  TRY(tmp.alloc(&bptr, (int64_t)nparts + 1));
  TRY(tmp.alloc(&bcol, ncand));
  TRY(tmp.alloc(&bperm, ncand));
  TRY(tmp.alloc(&gfirst, ncand + 1));
  TRY(tmp.alloc(&goff, (int64_t)nparts + 1));
  launch_col_parts(st, n, M.trowptr, M.trow, qptr, qpart, c->P.part, cptr, cpart);
  TRY(S.sort(n, nparts, ncand, cptr, cpart, bptr, bcol, bperm));
  gamma = cpart;                           // read no more
  TRY(S.distinct(nparts, ncand, bptr, bcol, gfirst, gamma, goff));
  const size_t row = ((size_t)nparts + 1) * sizeof(int32_t);
  LSQ2L_HIP_TRY(read(pptr, row, 0));
  LSQ2L_HIP_TRY(read(xoff, row, row));
  LSQ2L_HIP_TRY(read(goff, row, 2 * row));
  LSQ2L_HIP_TRY(hipStreamSynchronize(st));
  const int32_t *hp = back.p, *hx = hp + nparts + 1, *hg = hx + nparts + 1;
  const int64_t ng = hg[nparts];
  H.nparts = nparts;
  H.subs.assign((size_t)nparts, SubDesc{});
  int64_t omega_off = 0, loc_off = 0, tile_base = 0, g_off = 0;
  for (int32_t i = 0; i < nparts; ++i) {
    SubDesc& d = H.subs[i];
    d.nI = hp[i + 1] - hp[i];
    if (d.nI == 0) {
      set_error("part " + std::to_string(i) + " is empty");
      return LSQ2L_EINVAL;
    }
    d.nG = hg[i + 1] - hg[i];
    d.nIp = (d.nI + TS - 1) / TS * TS;
    d.nGp = (d.nG + TS - 1) / TS * TS;
    d.np = d.nIp + d.nGp;
    d.ntiles = d.np / TS;
    d.ntI = d.nIp / TS;
    d.nXi = hx[i + 1] - hx[i];
    d.seg = seg_of_part[i];
    d.id = i;
    d.omega_off = omega_off; omega_off += d.nI + d.nG;
    d.xi_off = hx[i];
    d.loc_off = loc_off; loc_off += d.np;
    d.tile_base = tile_base; tile_base += d.ntiles;
    d.dinv_off = d.tile_base * TT;
    d.g_off = g_off; g_off += (int64_t)d.nGp * d.nGp;
  }
  if (loc_off >= (int64_t)1 << 31) { set_error("local index space exceeds 2^31"); return LSQ2L_EINVAL; }
  H.total_loc = loc_off;
  H.total_tiles = tile_base;
  H.total_dinv = tile_base * TT;
  H.total_g = g_off;
  // Omega_i, the tile envelopes and their offsets; the descriptors are
  // uploaded twice, first without fac_off
  int64_t* stored = nullptr;
  SubDesc* dsub = nullptr;
  PinnedArray<SubDesc> hsub;
  PinnedArray<int64_t> hstored;
  TRY(hsub.alloc(nparts));
  TRY(hstored.alloc(nparts));
  TRY(tmp.alloc(&stored, nparts));
  TRY(c->dalloc(&dsub, nparts));
  TRY(c->dalloc(&c->P.omega, omega_off));
  TRY(c->dalloc(&c->P.tileF, tile_base));
  TRY(c->dalloc(&c->P.tileOff, tile_base));
  std::copy(H.subs.begin(), H.subs.end(), hsub.p);
  LSQ2L_HIP_TRY(hipMemcpyAsync(dsub, hsub.p, nparts * sizeof(SubDesc), hipMemcpyHostToDevice, st));
  launch_plan_omega(st, nparts, dsub, pptr, pcols, goff, gamma, c->P.omega, c->P.tileF);
  launch_plan_envelope(st, qptr, qpart, M, owner, dsub, goff, gamma, c->P.tileF);
  launch_tile_offsets(st, nparts, dsub, c->P.tileF, c->P.tileOff, stored);
  LSQ2L_HIP_TRY(hipMemcpyAsync(hstored.p, stored, nparts * sizeof(int64_t), hipMemcpyDeviceToHost, st));
  // inverse overlap map, and the pairs of parts that share rows
  int32_t *optr = nullptr, *opart = nullptr, *operm = nullptr, *pcnt = nullptr;
  TRY(tmp.alloc(&optr, (int64_t)n + 1));
  TRY(tmp.alloc(&opart, ng));
  TRY(tmp.alloc(&operm, ng));
  TRY(tmp.alloc(&pcnt, nx + 1));
  TRY(c->dalloc(&c->P.own_ptr, (int64_t)n + 1));
  TRY(c->dalloc(&c->P.own_pos, (int64_t)n + ng));
  TRY(S.sort(nparts, n, ng, goff, gamma, optr, opart, operm));
  launch_own_maps(st, n, c->P.part, c->P.locown, dsub, goff, optr, opart, operm, c->P.own_ptr, c->P.own_pos);
  TRY(keep.alloc(&out.pairs, npairs));
  launch_pair_count(st, nx, xi, qperm, qptr, pcnt);
  TRY(S.scan(nx + 1, pcnt));
  launch_pair_fill(st, nx, qperm, qpart, xoff, pcnt, out.pairs);
  LSQ2L_HIP_TRY(hipStreamSynchronize(st));
  LSQ2L_HIP_TRY(hipGetLastError());
  int64_t fac = 0;
  for (int32_t i = 0; i < nparts; ++i) {
    H.subs[i].fac_off = fac * TT;
    fac += hstored.p[i];
  }
  H.total_fac = fac * TT;
  c->P.subs = dsub;
  std::copy(H.subs.begin(), H.subs.end(), hsub.p);
  LSQ2L_HIP_TRY(hipMemcpyAsync(dsub, hsub.p, nparts * sizeof(SubDesc), hipMemcpyHostToDevice, st));
  LSQ2L_HIP_TRY(hipStreamSynchronize(st));
  out.npairs = npairs;
  out.done = true;
  return LSQ2L_OK;
}

lsq2l_status row_order_device(lsq2l_ctx* c, Scratch& tmp, int32_t* perm, int32_t* prp) {
  const hipStream_t st = c->st;
  const DevMatrix& M = c->M;
  Sorter S{st, tmp};
  int32_t *iota = nullptr, *key = nullptr, *kptr = nullptr, *again = nullptr;
  TRY(tmp.alloc(&iota, (int64_t)M.m + 1));
  TRY(tmp.alloc(&key, M.m));
  TRY(tmp.alloc(&kptr, (int64_t)M.n + 2));
  TRY(tmp.alloc(&again, M.m));
  launch_iota(st, (int64_t)M.m + 1, iota);
  launch_row_keys(st, M.m, M.n, M.rowptr, M.colind, key);
  TRY(S.sort(M.m, M.n + 1, M.m, iota, key, kptr, perm, again));
  launch_perm_len(st, M.m, perm, M.rowptr, prp);
  return S.scan((int64_t)M.m + 1, prp);
}

}  // namespace lsq2l
