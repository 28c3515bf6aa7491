// The cache of device blocks on a stubbed HIP allocator of bounded size: an
// allocation that fails at first and succeeds once the cache is empty leaves no
// error behind (kernel launches are checked with hipGetLastError), one that fails
// for good returns LSQ2L_ENOMEM, and every block is given back.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <string>

#include "../../paper_2107_09006_amd/csrc/ctx.hpp"
using namespace lsq2l;
#define CHECK(c, ...) do { if (!(c)) { fprintf(stderr, "FAIL %s:%d: ", __FILE__, __LINE__); fprintf(stderr, __VA_ARGS__); fprintf(stderr, "\n"); exit(1); } } while (0)

static const size_t MiB = (size_t)1 << 20, CARD = 1024 * MiB;
static size_t in_use = 0;
static char* next_addr = (char*)0x10000000000;
static std::map<void*, size_t> live;
static hipError_t last = hipSuccess;

extern "C" {
hipError_t hipMalloc(void** p, size_t bytes) {
  if (in_use + bytes > CARD) return last = hipErrorOutOfMemory;
  *p = next_addr;
  next_addr += bytes;
  live[*p] = bytes;
  in_use += bytes;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  CHECK(live.count(p), "free of a block that is not there");
  in_use -= live[p];
  live.erase(p);
  return hipSuccess;
}
hipError_t hipGetLastError(void) { const hipError_t e = last; last = hipSuccess; return e; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned) { *p = std::malloc(bytes); return hipSuccess; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stub"; }
}
namespace lsq2l {
static std::string message;
void set_error(const std::string& msg) { message = msg; }
}  // namespace lsq2l

int main() {
  void *a = nullptr, *b = nullptr;
  size_t na = 0, nb = 0;
  int dev = -1;
  CHECK(device_block(&a, 700 * MiB, &na, &dev) == LSQ2L_OK && a && na >= 700 * MiB && dev == 0, "first block");
  cache_give(a, na, dev);
  CHECK(live.size() == 1, "a block given back stays cached");
  CHECK(device_block(&a, 650 * MiB, &na, &dev) == LSQ2L_OK && live.size() == 1, "taken from the cache");
  cache_give(a, na, dev);
  // does not fit beside the cached block
  CHECK(device_block(&b, 400 * MiB, &nb, &dev) == LSQ2L_OK && b, "the retry after the cache is released");
  CHECK(live.size() == 1 && in_use == nb, "the cached block is gone");
  CHECK(hipGetLastError() == hipSuccess, "an allocation that succeeded leaves an error behind");
  void* c = nullptr;
  size_t nc = 0;
  CHECK(device_block(&c, 2 * CARD, &nc, &dev) == LSQ2L_ENOMEM && !c, "an allocation above the card");
  CHECK(message.find("failed") != std::string::npos, "its message");
  CHECK(hipGetLastError() == hipSuccess, "a failure that was reported leaves an error behind");
  cache_give(b, nb, dev);
  cache_release();
  CHECK(live.empty() && in_use == 0, "everything given back");
  // a handle's memory back to a mark: own blocks, arena chunks begun since, and
  // the place in the chunk that was open
  lsq2l_ctx& h = *new lsq2l_ctx();
  int32_t *x = nullptr, *y = nullptr, *z = nullptr, *again = nullptr;
  CHECK(h.dalloc(&x, 1000) == LSQ2L_OK, "from the arena");
  const size_t at_mark = in_use;
  const lsq2l_ctx::Mark k = h.mark();
  CHECK(h.dalloc(&y, 1000) == LSQ2L_OK && h.dalloc(&z, (int64_t)100 * MiB / 4) == LSQ2L_OK, "own block");
  for (int q = 0; q < 6; ++q) CHECK(h.dalloc(&z, (int64_t)60 * MiB / 4) == LSQ2L_OK, "a second chunk");
  CHECK(in_use > at_mark + 100 * MiB + 256 * MiB, "a block and a chunk more");
  h.rollback(k);
  cache_release();
  CHECK(in_use == at_mark, "given back to the mark");
  CHECK(h.dalloc(&again, 1000) == LSQ2L_OK && again == y, "the arena goes on at the mark");
  // an array of its own goes back alone; one at the start of a chunk does not
  // take the chunk with it
  int32_t *own = nullptr, *first = nullptr;
  CHECK(h.dalloc(&own, (int64_t)100 * MiB / 4) == LSQ2L_OK, "own block");
  for (int q = 0; q < 5; ++q) CHECK(h.dalloc(&first, (int64_t)60 * MiB / 4) == LSQ2L_OK, "a chunk's pieces");
  CHECK(live.count(first) == 1, "the last piece starts a chunk");
  const size_t with_own = in_use;
  h.give_back(own);
  h.give_back(first);
  cache_release();
  CHECK(!own && !first && with_own - in_use >= 100 * MiB && with_own - in_use < 200 * MiB, "one block given back");
  printf("OK\n");
  return 0;
}
