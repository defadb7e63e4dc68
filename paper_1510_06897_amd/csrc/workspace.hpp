// Device memory kept between calls: large work spaces and link fields.
//
// The device's stream-ordered pool does not keep them: whatever its release threshold, it gives free blocks
// back at any hipFree and at most calls of hipFreeAsync (a free 4 GB block was gone when the next, of 64 MB,
// was freed), and memory that was just given back is slow to map again (23 GB: 0.6 s).  A loop of handle,
// smearing, chain rule, force and sign function on 16^3 x 32 in FP64 takes 12.9 ms a step, 13.2 at most,
// with its blocks kept here; from the pool single steps took up to 1.4 s.
// Blocks of 16 MB and more are therefore kept here.  A block belongs to one user at a time; when it is
// given back an event marks the work that still uses it, and its next user's stream waits for that
// event, so blocks pass between streams and threads safely.  A block that another stream's work still
// uses is passed over while the library may have more memory, so that independent streams overlap.  At
// most an eighth of the device's memory is kept (least recently used freed first), and a block that 1024
// later returns did not need is freed.  Everything kept, and what the pool holds, goes back when any
// allocation of the library runs out of memory (with_room) and when the program asks for it (release):
// other allocators of the process, torch's among them, cannot reach it.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <vector>

namespace ovl {

constexpr size_t kKeepBlock = (size_t)16 << 20;  // smallest block kept
constexpr size_t kGrain = (size_t)2 << 20;       // block sizes are multiples of this
constexpr uint64_t kKeepReturns = 1024;

struct Block {
  void *p = nullptr;
  size_t bytes = 0;
  hipEvent_t evt = nullptr;  // (null: never kept) recorded at the last return, unless the device was idle then
  bool pending = false;      // evt may still have to be waited for
  hipStream_t stream = nullptr;  // where evt was recorded
  int dev = -1;
  uint64_t stamp = 0;
};

class BlockCache {
 public:
  // a block of at least `bytes` on the current device, usable in stream order on s
  hipError_t take(size_t bytes, hipStream_t s, Block &out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    bool more = false;  // another block is within the limit
    if (find(dev, bytes, s, false, out, &more) || (!more && find(dev, bytes, s, true, out))) return use(out, s);
    const Relaxed relaxed;
    Block b;
    b.bytes = (bytes + kGrain - 1) / kGrain * kGrain;
    b.dev = dev;
    e = hipMalloc(&b.p, b.bytes);
    if (e == hipErrorOutOfMemory) {
      (void)hipGetLastError();
      if (find(dev, bytes, s, true, out)) return use(out, s);
      release();
      e = hipMalloc(&b.p, b.bytes);
    }
    if (e != hipSuccess) return e;
    e = hipEventCreateWithFlags(&b.evt, hipEventDisableTiming);
    if (e != hipSuccess) {
      (void)hipFree(b.p);
      return e;
    }
    count(dev, b.bytes, true);
    out = b;
    return e;
  }

  // Memory of a handle made on stream s.  Below kKeepBlock it is allocated and freed as it is needed, and
  // so it is while s is captured: a kept block would make the capture wait on an event outside it.
  hipError_t take_handle(size_t bytes, hipStream_t s, Block &out) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    hipError_t e = hipStreamIsCapturing(s, &cap);
    if (e != hipSuccess) return e;
    if (bytes >= kKeepBlock && cap == hipStreamCaptureStatusNone) return take(bytes, s, out);
    e = hipGetDevice(&out.dev);
    if (e == hipSuccess) e = with_room([&] { return hipMalloc(&out.p, bytes); });
    if (e != hipSuccess) out = Block();
    else out.bytes = bytes;
    return e;
  }

  // Gives every kept block of the current device and the free memory of its stream-ordered pool back to
  // the device.
  void release() {
    int dev = 0;
    hipMemPool_t pool;
    if (hipGetDevice(&dev) == hipSuccess) {
      trim(dev, 0);
      const Relaxed relaxed;
      if (hipDeviceGetDefaultMemPool(&pool, dev) == hipSuccess) (void)hipMemPoolTrimTo(pool, 0);
    }
    (void)hipGetLastError();
  }

  // alloc(), and once more with everything kept given back if the device was out of memory
  template <class F>
  hipError_t with_room(F alloc) {
    const hipError_t e = alloc();
    if (e != hipErrorOutOfMemory) return e;
    (void)hipGetLastError();
    release();
    return alloc();
  }

  // hand a block back; s: the stream its last user worked on (other users' work has ended)
  void give(Block &b, hipStream_t s) {
    if (!b.p) return;
    if (!b.evt || hipEventRecord(b.evt, s) != hipSuccess) {
      (void)hipGetLastError();
      drop(b);
      return;
    }
    b.pending = true;
    b.stream = s;
    keep(b);
  }

  // hand back the block of a handle that ends; its work may be on any stream of the block's device, so
  // the device has to be idle.  Where that wait is refused (some stream is captured), and for a block that
  // is never kept, the block is freed instead: hipFree waits by itself.
  void retire(Block &b) {
    if (!b.p) return;
    const int dev = b.dev;
    int cur = dev;
    (void)hipGetDevice(&cur);
    if (cur != dev) (void)hipSetDevice(dev);
    if (hipDeviceSynchronize() == hipSuccess && b.evt) {
      b.pending = false;
      keep(b);
    } else {
      (void)hipGetLastError();
      drop(b);
    }
    if (cur != dev) (void)hipSetDevice(cur);
  }

 private:
  void keep(Block &b) {
    const int dev = b.dev;
    try {
      std::lock_guard<std::mutex> lk(mu_);
      b.stamp = ++clock_;
      free_.push_back(b);
    } catch (...) {  // no host memory to remember it by
      drop(b);
      return;
    }
    b = Block();
    trim(dev, limit(dev));
  }
  // Allocation and release are not stream operations: they leave a capture of another stream alone.
  struct Relaxed {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    Relaxed() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~Relaxed() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
  };
  void drop(Block &b) {
    const Relaxed relaxed;
    if (b.p && b.evt) count(b.dev, b.bytes, false);
    if (b.evt) (void)hipEventDestroy(b.evt);
    if (b.p) (void)hipFree(b.p);  // waits for the work that uses it
    (void)hipGetLastError();
    b = Block();
  }
  // a kept block in stream order on s
  hipError_t use(Block &b, hipStream_t s) {
    const hipError_t e = b.pending ? hipStreamWaitEvent(s, b.evt, 0) : hipSuccess;
    if (e != hipSuccess) drop(b);
    return e;
  }
  // the smallest kept block that fits: one whose work has ended or was on s, or (any) one to wait for;
  // *more: whether a block of `bytes` on top of all that exist stays within the limit
  bool find(int dev, size_t bytes, hipStream_t s, bool any, Block &out, bool *more = nullptr) {
    const size_t most = limit(dev);
    const Relaxed relaxed;
    std::lock_guard<std::mutex> lk(mu_);
    size_t best = free_.size();
    for (size_t i = 0; i < free_.size(); ++i) {
      Block &b = free_[i];
      if (b.dev != dev || b.bytes < bytes || b.bytes - bytes > std::max(bytes / 2, kGrain)) continue;
      if (!any && b.pending && b.stream != s) {
        if (hipEventQuery(b.evt) != hipSuccess) {
          (void)hipGetLastError();
          continue;
        }
        b.pending = false;
      }
      if (best == free_.size() || b.bytes < free_[best].bytes) best = i;
    }
    if (more) *more = dev >= 0 && dev < 64 && owned_[dev] + bytes <= most;
    if (best == free_.size()) return false;
    out = free_[best];
    free_.erase(free_.begin() + best);
    return true;
  }
  void count(int dev, size_t bytes, bool up) {
    std::lock_guard<std::mutex> lk(mu_);
    if (dev >= 0 && dev < 64) owned_[dev] = up ? owned_[dev] + bytes : owned_[dev] - bytes;
  }
  size_t limit(int dev) {
    if (dev < 0 || dev >= 64) return 0;
    std::call_once(once_[dev], [&] {
      if (hipDeviceTotalMem(&total_[dev], dev) != hipSuccess) total_[dev] = 0;
    });
    return total_[dev] / 8;
  }
  void trim(int dev, size_t most) {
    for (;;) {
      Block b;
      {
        std::lock_guard<std::mutex> lk(mu_);
        size_t held = 0, old = free_.size();
        for (size_t i = 0; i < free_.size(); ++i)
          if (free_[i].dev == dev) {
            held += free_[i].bytes;
            if (old == free_.size() || free_[i].stamp < free_[old].stamp) old = i;
          }
        if (old == free_.size() || (held <= most && clock_ - free_[old].stamp <= kKeepReturns)) return;
        b = free_[old];
        free_.erase(free_.begin() + old);
      }
      drop(b);
    }
  }

  std::mutex mu_;
  std::vector<Block> free_;
  uint64_t clock_ = 0;
  size_t owned_[64] = {};  // bytes of a device's blocks, kept and in use
  std::once_flag once_[64];
  size_t total_[64] = {};
};

// never destroyed: handles may outlive static destruction, and the process's end frees the memory
inline BlockCache &block_cache() {
  static BlockCache *c = new BlockCache();
  return *c;
}

}  // namespace ovl
