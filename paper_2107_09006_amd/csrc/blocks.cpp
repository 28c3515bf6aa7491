// Memory that outlives a handle: the cache of device blocks and the pool of
// pinned host buffers, with the allocations that draw on them.
#include <mutex>
#include <string>
#include <vector>

#include "ctx.hpp"

namespace lsq2l {
namespace {

// Device blocks of destroyed handles, kept for later handles on the same
// device: a setup allocates gigabytes in blocks of hundreds of megabytes,
// and allocating or releasing a block of that size costs a sizeable fraction
// of a millisecond.  A request takes the smallest cached block of its device
// that is at least as large and at most a quarter larger.  At most
// CACHE_LIMIT bytes stay cached; lsq2l_release_cache() frees them all, and an
// allocation that fails frees them and tries once more.
struct BlockCache {
  struct Block { void* p; size_t bytes; int dev; };
  static constexpr size_t CACHE_LIMIT = (size_t)32 << 30;
  std::mutex mu;
  std::vector<Block> blocks;
  size_t held = 0;
  void* take(size_t bytes, int dev, size_t* got) {
    std::lock_guard<std::mutex> g(mu);
    int best = -1;
    for (int i = 0; i < (int)blocks.size(); ++i) {
      const Block& b = blocks[i];
      if (b.dev != dev || b.bytes < bytes || b.bytes > bytes + bytes / 4) continue;
      if (best < 0 || b.bytes < blocks[best].bytes) best = i;
    }
    if (best < 0) return nullptr;
    void* p = blocks[best].p;
    *got = blocks[best].bytes;
    held -= *got;
    blocks.erase(blocks.begin() + best);
    return p;
  }
  // the caller has synchronized the work that used the block
  void give(void* p, size_t bytes, int dev) {
    std::lock_guard<std::mutex> g(mu);
    if (held + bytes > CACHE_LIMIT) {
      int cur = 0;
      (void)hipGetDevice(&cur);
      (void)hipSetDevice(dev);
      (void)hipFree(p);
      (void)hipSetDevice(cur);
      return;
    }
    blocks.push_back({p, bytes, dev});
    held += bytes;
  }
  void release() {
    std::lock_guard<std::mutex> g(mu);
    int cur = 0;
    (void)hipGetDevice(&cur);
    for (const Block& b : blocks) {
      (void)hipSetDevice(b.dev);
      (void)hipFree(b.p);
    }
    (void)hipSetDevice(cur);
    blocks.clear();
    held = 0;
  }
};

// never destroyed: device memory goes back with the process
BlockCache& block_cache() {
  static BlockCache* bc = new BlockCache();
  return *bc;
}

// Pinned host buffers for the copies setup reads back from the device (A's
// pattern, A^T's pattern) and stages its uploads through, kept for later
// setups: a pageable copy runs at a sixth of the pinned rate, and pinning
// fresh memory costs more than the copy.  At most PINNED_LIMIT bytes stay
// cached.
struct PinnedPool {
  struct Buf { void* p; size_t bytes; };
  static constexpr size_t PINNED_LIMIT = (size_t)4 << 30;
  std::mutex mu;
  std::vector<Buf> bufs;
  size_t held = 0;
  void* take(size_t bytes, size_t* got) {
    {
      std::lock_guard<std::mutex> g(mu);
      int best = -1;
      for (int i = 0; i < (int)bufs.size(); ++i)
        if (bufs[i].bytes >= bytes && bufs[i].bytes <= 2 * bytes &&
            (best < 0 || bufs[i].bytes < bufs[best].bytes))
          best = i;
      if (best >= 0) {
        void* p = bufs[best].p;
        *got = bufs[best].bytes;
        held -= *got;
        bufs.erase(bufs.begin() + best);
        return p;
      }
    }
    void* p = nullptr;
    if (hipHostMalloc(&p, bytes, hipHostMallocDefault) != hipSuccess) {
      (void)hipGetLastError();
      return nullptr;
    }
    *got = bytes;
    return p;
  }
  void give(void* p, size_t bytes) {
    std::lock_guard<std::mutex> g(mu);
    if (held + bytes > PINNED_LIMIT) {
      (void)hipHostFree(p);
      return;
    }
    bufs.push_back({p, bytes});
    held += bytes;
  }
  void release() {
    std::lock_guard<std::mutex> g(mu);
    for (const Buf& b : bufs) (void)hipHostFree(b.p);
    bufs.clear();
    held = 0;
  }
};

PinnedPool& pinned_pool() {
  static PinnedPool* pp = new PinnedPool();
  return *pp;
}

}  // namespace

void* cache_take(size_t bytes, int dev, size_t* got) { return block_cache().take(bytes, dev, got); }
void cache_give(void* p, size_t bytes, int dev) { block_cache().give(p, bytes, dev); }
void cache_release() { block_cache().release(); }
void* pinned_take(size_t bytes, size_t* got) { return pinned_pool().take(bytes, got); }
void pinned_give(void* p, size_t bytes) { pinned_pool().give(p, bytes); }
void pinned_release() { pinned_pool().release(); }

// host arrays of the planner: from 1 MiB up in the pinned pool (whole MiB),
// smaller ones from the heap
void* host_block_take(size_t bytes, size_t* got) {
  constexpr size_t MiB = (size_t)1 << 20;
  if (bytes < MiB) {
    *got = bytes;
    return std::malloc(bytes);
  }
  return pinned_take((bytes + MiB - 1) / MiB * MiB, got);
}
void host_block_give(void* p, size_t bytes) {
  if (bytes < ((size_t)1 << 20)) std::free(p);
  else pinned_give(p, bytes);
}

}  // namespace lsq2l

using namespace lsq2l;

lsq2l_status lsq2l::device_block(void** v, size_t bytes, size_t* got, int* dev, bool exact) {
  *v = nullptr;
  LSQ2L_HIP_TRY(hipGetDevice(dev));
  // eight sizes per power of two: problems that are alike ask for the same
  // blocks, and a setup on new inputs finds what an earlier one left (with
  // the sizes as asked, irregular matrices of 1e6 columns took 182 ms instead
  // of 96 on new inputs)
  size_t step = (size_t)1 << 20;
  while (step * 16 <= bytes) step *= 2;
  if (!exact) bytes = (bytes + step - 1) / step * step;
  if ((*v = cache_take(bytes, *dev, got)) != nullptr) return LSQ2L_OK;
  // a failure is cleared, or the next launch's check would report it
  hipError_t e = hipMalloc(v, bytes);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    cache_release();
    e = hipMalloc(v, bytes);
  }
  if (e != hipSuccess) {
    (void)hipGetLastError();
    *v = nullptr;
    set_error("device allocation of " + std::to_string(bytes) + " bytes failed: " + hipGetErrorString(e));
    return LSQ2L_ENOMEM;
  }
  *got = bytes;
  return LSQ2L_OK;
}

lsq2l_status lsq2l_ctx::raw_alloc(void** v, size_t bytes) {
  DevBlock b{};
  TRY(device_block(&b.p, bytes, &b.bytes, &b.dev, lean));
  dev_allocs.push_back(b);
  *v = b.p;
  return LSQ2L_OK;
}
