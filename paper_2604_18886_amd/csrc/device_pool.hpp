// Device memory of the library's objects.  Plain C++: the runtime's calls come
// in as `Api`, so that the pool's decisions can be checked on the host.
#pragma once

#include <cstddef>
#include <cstdint>
#include <iterator>
#include <list>
#include <mutex>
#include <new>

namespace mfmg {

// hipMalloc and hipFree map, clear and unmap pages: a program that rebuilds
// its octree and hierarchy every step (4 GB of them at 26.3M leaves) spent most
// of the rebuild in them (123 ms, of which the kernels are 5; 7.3 ms with this
// pool).  Freed blocks are kept per device and handed out again by size, which
// is rounded up by less than an eighth.
//
// Kept blocks are out of reach of the process's other allocators, so they are
// bounded: at most kMaxBytes, and beyond kAsk at most a quarter of what the
// device has free besides (the least recently freed go back to the driver first); a block not
// asked for within kMaxAge frees goes back too, and everything does when an
// allocation fails or on request (release).
//
// A block may be handed to any stream and thread, so it is kept only once the
// device has finished its work (as hipFree waited).  Where that wait fails (it
// is refused while the process captures a stream) the work may still be
// running: the block is parked, and kept after a wait that succeeds.
//
// Api, all on the current device: Status alloc(bytes, void **), bool
// out_of_memory(Status) (which also clears the error), bool free(void *) (false:
// refused, the block stays), bool wait() (for everything queued; false: it may
// still run), bool available(size_t *) (free bytes of the device).
template <class Api>
class DevicePool {
 public:
  using Status = typename Api::Status;
  static constexpr size_t kMaxBytes = size_t(8) << 30;
  static constexpr uint64_t kMaxAge = 512;
  static constexpr size_t kAsk = size_t(1) << 30;

  // A multiple of 512, more than bytes by less than an eighth of it from 4 KiB on.
  static size_t rounded(size_t bytes) {
    size_t step = 512;
    while (step * 16 < bytes) step *= 2;
    return (bytes + step - 1) / step * step;
  }

  // bytes: a rounded size
  Status get(size_t bytes, void **out) {
    {
      std::lock_guard<std::mutex> lock(mu_);
      for (auto it = kept_.rbegin(); it != kept_.rend(); ++it)
        if (it->bytes == bytes) {
          *out = it->p;
          held_ -= bytes;
          kept_.erase(std::next(it).base());
          return Status{};
        }
    }
    Status e = Api::alloc(bytes, out);
    if (Api::out_of_memory(e)) {
      settle();
      std::lock_guard<std::mutex> lock(mu_);
      trim(0, 0);
      e = Api::alloc(bytes, out);
    }
    return e;
  }

  // drained: the work that uses the block is known to have finished
  void put(void *p, size_t bytes, bool drained) {
    std::list<Block> one;
    try {
      one.push_back(Block{p, bytes, 0});
    } catch (const std::bad_alloc &) {
      if (drained || Api::wait()) (void)Api::free(p);
      return;
    }
    if (!drained) {
      {
        std::lock_guard<std::mutex> lock(mu_);
        parked_.splice(parked_.end(), one);
      }
      settle();
      return;
    }
    std::lock_guard<std::mutex> lock(mu_);
    keep(one);
  }

  // as put, but the block goes back to the driver
  void drop(void *p, size_t bytes, bool drained) {
    if (!(drained || Api::wait()) || !Api::free(p)) put(p, bytes, false);
  }

  // Takes the bound on kept blocks from what the device has free now.  Asking
  // takes some 10 microseconds (a small object is made and destroyed in 25, the
  // three of 26.3M leaves in 2,700), so not per block: called after an object's
  // are back, and only once kAsk more have come back.
  void rebound() {
    {
      std::lock_guard<std::mutex> lock(mu_);
      if (back_ < kAsk) return;
      back_ = 0;
    }
    size_t n = 0;
    if (!Api::available(&n)) return;
    std::lock_guard<std::mutex> lock(mu_);
    most_ = n / 4 < kMaxBytes ? n / 4 : kMaxBytes;
    trim(most_, 0);
  }

  // Gives every kept block back to the driver.
  void release() {
    bool late = false;
    {
      std::lock_guard<std::mutex> lock(mu_);
      late = !parked_.empty();
    }
    if (late) settle();
    std::lock_guard<std::mutex> lock(mu_);
    trim(0, 0);
  }

  // Waits for the device; true if it has finished, and then the blocks parked
  // before the wait are kept.
  bool settle() {
    std::list<Block> late;
    {
      std::lock_guard<std::mutex> lock(mu_);
      late.swap(parked_);
    }
    const bool done = Api::wait();
    std::lock_guard<std::mutex> lock(mu_);
    if (done) keep(late);
    else parked_.splice(parked_.end(), late);
    return done;
  }

 private:
  struct Block {
    void *p;
    size_t bytes;
    uint64_t when;
  };
  void keep(std::list<Block> &blocks) {
    for (Block &b : blocks) {
      b.when = ++frees_;
      held_ += b.bytes;
      back_ += b.bytes;
    }
    kept_.splice(kept_.end(), blocks);
    trim(most_, frees_ > kMaxAge ? frees_ - kMaxAge : 0);
  }
  void trim(size_t most, uint64_t oldest) {
    while (!kept_.empty() && (held_ > most || kept_.front().when < oldest)) {
      if (!Api::free(kept_.front().p)) return;
      held_ -= kept_.front().bytes;
      kept_.pop_front();
    }
  }
  std::mutex mu_;
  std::list<Block> kept_;    // least recently freed first
  std::list<Block> parked_;  // freed, their work not known to have finished
  size_t held_ = 0;          // bytes in kept_
  size_t most_ = kMaxBytes;  // and their bound
  size_t back_ = 0;          // bytes put back since it was taken
  uint64_t frees_ = 0;
};

}  // namespace mfmg
