// Checks of the device memory pool's decisions on a stand-in device that counts
// its blocks.  Usage: device_pool_check CASE; exits with 0 when it holds.
#include <cstdio>
#include <cstring>
#include <map>
#include <vector>

#include "device_pool.hpp"

struct Device {
  using Status = int;  // 0 ok, 1 out of memory
  static std::map<void *, size_t> live;
  static size_t used, capacity, next;
  static bool busy;  // waits and frees are refused
  static int waits, asked;
  static int alloc(size_t bytes, void **out) {
    if (used + bytes > capacity) return 1;
    *out = reinterpret_cast<void *>(next += 4096);
    live[*out] = bytes;
    used += bytes;
    return 0;
  }
  static bool out_of_memory(int e) { return e == 1; }
  static bool free(void *p) {
    if (busy) return false;
    used -= live.at(p);
    live.erase(p);
    return true;
  }
  static bool available(size_t *bytes) {
    ++asked;
    *bytes = capacity - used;
    return true;
  }
  static bool wait() {
    ++waits;
    return !busy;
  }
};
std::map<void *, size_t> Device::live;
size_t Device::used = 0, Device::capacity = size_t(1) << 40, Device::next = 0;
bool Device::busy = false;
int Device::waits = 0, Device::asked = 0;

using Pool = mfmg::DevicePool<Device>;

#define CHECK(x)                                              \
  do {                                                        \
    if (!(x)) {                                               \
      std::printf("%s:%d: %s\n", __FILE__, __LINE__, #x);     \
      return 1;                                               \
    }                                                         \
  } while (0)

// A block whose work may still be running is handed to nobody, also not by an
// allocation that finds the device full, until a wait succeeds.
static int failed_wait() {
  Pool pool;
  const size_t n = Pool::rounded(size_t(1) << 20);
  void *a = nullptr, *b = nullptr, *c = nullptr;
  CHECK(pool.get(n, &a) == 0);
  Device::busy = true;
  pool.put(a, n, false);
  CHECK(Device::waits == 1);
  CHECK(pool.get(n, &b) == 0 && b != a);
  CHECK(Device::live.count(a));
  Device::capacity = Device::used;
  CHECK(pool.get(n, &c) == 1 && Device::live.count(a));
  pool.put(b, n, true);  // its own work has finished: kept at once
  CHECK(pool.get(n, &c) == 0 && c == b);
  CHECK(!pool.settle());
  Device::busy = false;
  CHECK(pool.get(n, &b) == 0 && !Device::live.count(a));  // full: parked block given back
  pool.put(b, n, false);
  CHECK(pool.get(n, &a) == 0 && a == b);  // waited for: kept
  Device::busy = true;
  pool.put(a, n, false);
  Device::busy = false;
  CHECK(pool.settle());
  CHECK(pool.get(n, &b) == 0 && b == a);
  return 0;
}

// Sizes are rounded up by less than an eighth (by less than 512 bytes below 4
// KiB), and a larger request never to less.
static int rounding() {
  size_t last = 0;
  for (int k = 0; k < 40; ++k)
    for (int step = 8; step < 16; ++step)
      for (int off = -1; off <= 1; ++off) {
        const size_t n = ((size_t(step) << k) >> 3) + size_t(off);
        if (n == 0 || n > (size_t(1) << 41)) continue;
        const size_t r = Pool::rounded(n);
        CHECK(r >= n && r % 512 == 0);
        CHECK(n < 4096 ? r - n < 512 : (r - n) * 8 < n);
        CHECK(Pool::rounded(r) == r);
        CHECK(off == -1 || r >= last);
        last = r;
      }
  return 0;
}

// A dropped block goes back at once, or waits with the parked ones.
static int dropped() {
  Pool pool;
  void *a = nullptr, *b = nullptr;
  CHECK(pool.get(4096, &a) == 0 && pool.get(4096, &b) == 0);
  pool.drop(a, 4096, true);
  CHECK(!Device::live.count(a));
  Device::busy = true;
  pool.drop(b, 4096, false);
  CHECK(Device::live.count(b));
  CHECK(pool.get(4096, &a) == 0 && a != b);
  Device::busy = false;
  pool.drop(a, 4096, false);
  CHECK(!Device::live.count(a));
  return 0;
}

constexpr size_t kMiB = size_t(1) << 20;

// Fills a pool with n kept blocks of the given size.
static int fill(Pool &pool, int n, size_t bytes, std::vector<void *> &p) {
  p.assign(size_t(n), nullptr);
  for (void *&q : p) CHECK(pool.get(bytes, &q) == 0);
  for (void *q : p) pool.put(q, bytes, true);
  return 0;
}

// At most kMaxBytes are kept; the least recently freed blocks go first.
static int most_kept() {
  Pool pool;
  std::vector<void *> p;
  CHECK(fill(pool, 40, 512 * kMiB, p) == 0);
  CHECK(Device::used == Pool::kMaxBytes);
  for (int i = 0; i < 40; ++i) CHECK(Device::live.count(p[size_t(i)]) == (i >= 24));
  return 0;
}

// A block not asked for within kMaxAge frees goes back.
static int ageing() {
  Pool pool;
  void *old = nullptr, *b = nullptr;
  CHECK(pool.get(2 * kMiB, &old) == 0);
  pool.put(old, 2 * kMiB, true);
  for (uint64_t i = 0; i < Pool::kMaxAge; ++i) {
    CHECK(Device::live.count(old));
    CHECK(pool.get(kMiB, &b) == 0);
    pool.put(b, kMiB, true);
  }
  CHECK(pool.get(kMiB, &b) == 0);
  pool.put(b, kMiB, true);
  CHECK(!Device::live.count(old) && Device::live.count(b));
  return 0;
}

// An allocation that finds the device full gets what is kept.
static int full_device() {
  Pool pool;
  std::vector<void *> p;
  Device::capacity = 8 * kMiB;
  CHECK(fill(pool, 8, kMiB, p) == 0);
  void *q = nullptr;
  CHECK(pool.get(8 * kMiB, &q) == 0);
  CHECK(pool.get(kMiB, &q) == 1);
  return 0;
}

// Others can have what is kept: once kAsk have come back at most a quarter of
// the free memory stays, and nothing after release (blocks whose free is refused
// do).
static int given_back() {
  Pool pool;
  std::vector<void *> p;
  Device::capacity = 4096 * kMiB;
  CHECK(fill(pool, 30, 32 * kMiB, p) == 0);
  pool.rebound();
  CHECK(Device::asked == 0 && Device::used == 960 * kMiB);
  CHECK(fill(pool, 60, 32 * kMiB, p) == 0);
  pool.rebound();  // 2176 MiB free: a quarter is 544 MiB
  CHECK(Device::asked == 1 && Device::used == 544 * kMiB);
  CHECK(fill(pool, 30, 32 * kMiB, p) == 0);
  CHECK(Device::used == 544 * kMiB);
  Device::busy = true;
  pool.release();
  CHECK(Device::used == 544 * kMiB);
  void *q = nullptr;
  CHECK(pool.get(32 * kMiB, &q) == 0 && Device::used == 544 * kMiB);
  pool.put(q, 32 * kMiB, false);  // parked
  Device::busy = false;
  pool.release();
  CHECK(Device::used == 0);
  return 0;
}

int main(int argc, char **argv) {
  const char *name = argc > 1 ? argv[1] : "";
  if (!std::strcmp(name, "failed_wait")) return failed_wait();
  if (!std::strcmp(name, "rounding")) return rounding();
  if (!std::strcmp(name, "dropped")) return dropped();
  if (!std::strcmp(name, "most_kept")) return most_kept();
  if (!std::strcmp(name, "ageing")) return ageing();
  if (!std::strcmp(name, "full_device")) return full_device();
  if (!std::strcmp(name, "given_back")) return given_back();
  std::printf("unknown case %s\n", name);
  return 2;
}
