// Host memory and copies of the transfers between the caller's memory and the
// device.
#pragma once

#include <algorithm>
#include <cstring>

#include "common.hpp"
#include "host_pool.hpp"

namespace gsmat {

// Host memory that large transfers go through: two parts, one worked on by the
// device while the host copies the other, and the tasks and reports of each.
// Per thread, 0.5 MiB until a transfer needs more, then 8.2 MiB, given back at
// the thread's end.
struct FetchArea {
  static constexpr size_t kSmall = 128 << 10, kLarge = 4 << 20;  // bytes per part
  char* p = nullptr;
  size_t part = 0;
  uint32_t* words(int i) { return (uint32_t*)(p + 2 * part) + i * kPackWords; }
  PackTask* tasks(int i) { return (PackTask*)(words(0) + 2 * kPackWords) + i * kPackGroups; }
  int32_t* rows(int i) { return (int32_t*)(p + i * part); }
  void reserve(size_t bytes) {
    const size_t want = bytes <= kSmall ? kSmall : kLarge;
    if (part >= want) return;
    release();
    const size_t all =
        2 * (want + sizeof(uint32_t) * kPackWords + sizeof(PackTask) * kPackGroups);
    GS_HIP(hipHostMalloc((void**)&p, all, hipHostMallocDefault));
    part = want;
    std::memset(words(0), 0, 2 * sizeof(uint32_t) * kPackWords);
  }
  void release() {
    if (p) (void)hipHostFree(p);
    p = nullptr;
    part = 0;
  }
  ~FetchArea() { release(); }
};
inline FetchArea& fetch_area() {
  thread_local FetchArea a;
  return a;
}

// A piece of a transfer, shared by the host pool: one thread copies 10 to 15
// GB/s, a quarter of the link.
inline void copy_host(char* to, const char* from, int64_t bytes) {
  constexpr int64_t kUnit = 64 << 10;
  const int64_t units = ceil_div(bytes, kUnit);
  host_parallel_for(units, 8, [&](int64_t lo, int64_t hi) {
    std::memcpy(to + lo * kUnit, from + lo * kUnit,
                (size_t)(std::min(hi * kUnit, bytes) - lo * kUnit));
  });
}
// Makes the next 32 MiB of [p, end), all of which is about to be written,
// present in memory; returns where it got to.  A piece of a fetch covers two
// large pages, which two threads would clear while the others wait for them;
// here each thread clears pages of its own (3 million rows of 4 columns: 2.9 ->
// 2.2 ms).
inline char* map_ahead(char* p, char* end) {
  constexpr int64_t kPage = 4096, kUnit = 2 << 20;
  char* const to = p + std::min<int64_t>(end - p, 16 * kUnit);
  host_parallel_for(ceil_div(to - p, kUnit), 1, [&](int64_t lo, int64_t hi) {
    for (char* a = p + lo * kUnit; a < std::min(to, p + hi * kUnit); a += kPage)
      *(volatile char*)a = 0;
  });
  return to;
}

}  // namespace gsmat
