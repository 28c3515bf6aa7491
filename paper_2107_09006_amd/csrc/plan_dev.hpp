// Device planner: the plan of plan_build, the overlap map of plan_maps and the
// order of row_order, formed on the GPU from the device copy of A.
#pragma once
#include "ctx.hpp"

namespace lsq2l {

// Device work space of a setup, from the block cache; given back by the
// destructor, after the stream has drained.
struct Scratch {
  hipStream_t st = nullptr;
  std::vector<lsq2l_ctx::DevBlock> blocks;
  explicit Scratch(hipStream_t s) : st(s) {}
  Scratch(const Scratch&) = delete;
  Scratch& operator=(const Scratch&) = delete;
  ~Scratch() { release(); }
  void release() {
    if (blocks.empty()) return;
    (void)hipStreamSynchronize(st);
    for (const auto& b : blocks) cache_give(b.p, b.bytes, b.dev);
    blocks.clear();
  }
  template <typename T>
  lsq2l_status alloc(T** p, int64_t count, bool exact = false) {
    lsq2l_ctx::DevBlock b{};
    lsq2l_status s = device_block(&b.p, (size_t)std::max<int64_t>(count, 1) * sizeof(T), &b.bytes, &b.dev, exact);
    if (s == LSQ2L_OK) blocks.push_back(b);
    *p = (T*)b.p;
    return s;
  }
};

// Work space of a transpose of nnz entries and n columns: what carries rows and
// values through the sort, or where that cannot be had the least (a third of it;
// rows and values are gathered then, see launch_transpose)
inline lsq2l_status transpose_space(Scratch& s, bool lean, int64_t nnz, int32_t n, char** temp, size_t* bytes) {
  *bytes = transpose_temp_bytes(nnz, n);
  if (!lean && s.alloc(temp, (int64_t)*bytes) == LSQ2L_OK) return LSQ2L_OK;
  *bytes = transpose_temp_least(nnz, n);
  return s.alloc(temp, (int64_t)*bytes, lean);
}

// From this many entries on the device plans: some thirty launches and six
// reads of counts.  Whole setups in ms, device / host planner, at three kinds of
// matrix: banded (125 columns per part), grid (20 x 20 per part), irregular (1,000):
//   4,000 -  7,000 entries   2.06 / 1.89   1.78 / 1.54    5.25 / 5.01
//   8,700 - 10,700           2.01 / 2.08   2.03 / 1.90   16.3  / 16.2
//  12,300 - 15,300           2.10 / 2.28   2.27 / 2.11    5.09 / 4.91
//  17,800 - 21,100           2.09 / 2.56   2.93 / 3.11    6.79 / 6.63
//  74,000 - 89,000           2.36 / 3.11   3.69 / 4.57   15.8  / 15.9
// The line lies where the first kind crosses; the others do at 16,000 and 80,000,
// with less than 5 % between the planners from 12,000 on.  Planning alone: 0.6
// (0.51) at 9,000 banded entries, 0.88 (2.3) at 3e5, 1.2 (6.9) at 3.8e6, 5.5 (16)
// at 3.3e7.
constexpr int64_t DEVICE_PLAN_NNZ = (int64_t)1 << 13;
// Longest row or column, and largest product of a shared row's length with its
// number of parts, that a few lanes walk one after the other: some milliseconds
// (the host planner's threads take such a row in less).
constexpr unsigned long long DEVICE_PLAN_LONGEST = 1 << 15;

struct DevicePlan {
  bool done = false;            // false: the host has to plan (see plan_build_device)
  int64_t npairs = 0;           // pairs of parts sharing a row
  int4* pairs = nullptr;        // in scratch given by the caller
  int64_t far_descents = 0;     // of row_order
};

// Fills c->H's sizes and offsets and c->P's omega, xi, locown, tileF, tileOff,
// subs, own_ptr and own_pos (c->P.part and A^T are there), with owner per
// entry of A (launch_entry_owner).  done stays false where the host planner is
// to take over: a row or column above DEVICE_PLAN_LONGEST, rows that so many
// parts share that the lists of candidates would be long (more than eight times
// the entries of A; the host needs no such lists), or work space short.
lsq2l_status plan_build_device(lsq2l_ctx* c, int32_t nparts, const std::vector<int32_t>& seg_of_part,
                               int2* owner, Scratch& keep, DevicePlan& out);

// The order of row_order on the device: perm and row pointer of the copy
lsq2l_status row_order_device(lsq2l_ctx* c, Scratch& tmp, int32_t* perm, int32_t* prp);

}  // namespace lsq2l
