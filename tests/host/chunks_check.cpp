// The cuts of a concatenated vector (make_chunks) for instances of every mixture
// of lengths: each chunk inside its instance, consecutive, together the whole
// vector; the number and order of an instance's chunks, its counters' slot, and
// the bound on their total.  No GPU is used.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <set>
#include <vector>

#include "../../paper_2107_09006_amd/csrc/kernels.hpp"
using namespace lsq2l;
#define CHECK(c, ...) do { if (!(c)) { fprintf(stderr, "FAIL %s:%d: ", __FILE__, __LINE__); fprintf(stderr, __VA_ARGS__); fprintf(stderr, "\n"); exit(1); } } while (0)

static void check(const std::vector<int64_t>& len, int64_t size, int64_t most) {
  std::vector<int64_t> seg(1, 0);
  for (int64_t l : len) seg.push_back(seg.back() + l);
  const std::vector<Chunk> c = make_chunks(seg, size, most);
  std::set<int32_t> slots;
  size_t at = 0;
  int64_t bound = 0;
  for (size_t s = 0; s < len.size(); ++s) {
    const int32_t n = c.at(at).n;
    CHECK(n >= 1 && n <= most && (n == most || (int64_t)n * size < len[s] + size || n == 1), "count of %zu", s);
    if (n > 1) CHECK(slots.insert(c[at].slot).second, "slot of %zu", s);
    int64_t pos = seg[s];
    for (int32_t k = 0; k < n; ++k, ++at) {
      const Chunk& q = c.at(at);
      CHECK(q.seg == (int32_t)s && q.k == k && q.n == n && q.slot == c[at - k].slot, "chunk %zu", at);
      CHECK(q.lo == pos && q.len >= 0 && pos + q.len <= seg[s + 1], "extent of %zu", at);
      CHECK(n == most || q.len <= size, "length of %zu", at);
      pos += q.len;
    }
    CHECK(pos == seg[s + 1], "instance %zu is covered", s);
    bound += 1 + len[s] / size;
  }
  CHECK(at == c.size() && (int64_t)at <= bound, "total");
  for (int32_t q : slots) CHECK(q >= 0 && q < (int32_t)slots.size(), "slots are numbered through");
}

int main() {
  std::mt19937_64 rng(5);
  std::vector<std::vector<int64_t>> sets = {{1}, {1024}, {1025}, {262144}, {262145}, {9000000}, {1000000000},
                                            {1, 1000000, 1}};
  sets.push_back(std::vector<int64_t>(5000, 3));
  sets.back()[2500] = 20000000;
  for (int t = 0; t < 200; ++t) {
    std::vector<int64_t> v(1 + rng() % 300);
    for (int64_t& x : v) x = 1 + rng() % ((uint64_t)1 << (rng() % 24));
    sets.push_back(v);
  }
  for (const auto& v : sets) {
    int64_t total = 0;
    for (int64_t x : v) total += x;
    const int64_t q = reduction_chunk(total);
    CHECK(q >= 1024 && (total + q - 1) / q <= RED_TOTAL, "chunk size of %lld", (long long)total);
    check(v, q, RED_BLOCKS);
    check(v, q, MDOT_BLOCKS);
    check(v, 1024, INT64_MAX);
  }
  printf("OK\n");
  return 0;
}
