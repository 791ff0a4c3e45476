// The block table of a KV fetch that allocates nothing (mma_kv_fetch_noalloc), on
// its way to the launch that needs it. Host code only; a CPU test calls it with
// launches of its own.
#ifndef MMA_NOALLOC_H_
#define MMA_NOALLOC_H_

#include <algorithm>
#include <vector>

#include "mma_engine.h"

namespace mma {

// The table of n blocks into the arguments a, behind the layer pointers, if it fits
// them; else into the scratch array by launches made through `launch`, chunk by chunk:
// no copy call and no staging buffer. sorted: by destination, as a pool in HBM is
// taken. Returns what a failed launch returned, or 0.
// Calls share nothing here, so one whose launches wait (a full queue) holds up no
// other. A table to be sorted that does not fit the arguments needs room for twice
// its entries, 1 MiB at most, which the thread keeps until it ends.
template <class Launch>
inline int noalloc_table(PoolArgs& a, uint64_t* scratch, const int32_t* host_slots, const int32_t* gpu_blocks,
                         uint32_t n, bool sorted, Launch launch) {
  const auto entry = [&](uint32_t i) {
    return static_cast<uint64_t>(static_cast<uint32_t>(host_slots[i])) |
           (static_cast<uint64_t>(static_cast<uint32_t>(gpu_blocks[i])) << 32);
  };
  if (a.layers + n <= kPoolWords) {
    uint64_t* const w = a.w + a.layers;
    for (uint32_t i = 0; i < n; ++i) w[i] = entry(i);
    a.words = a.layers + n;
    if (sorted) {
      uint64_t tmp[kPoolWords];
      sort_table(w, n, 32, tmp);
    }
    return 0;
  }
  static thread_local std::vector<uint64_t> room;
  if (sorted) {
    if (room.size() < 2ull * n) room.resize(2ull * n);
    for (uint32_t i = 0; i < n; ++i) room[i] = entry(i);
    sort_table(room.data(), n, 32, room.data() + n);
  }
  a.tab = scratch + kNoallocTabOffset / 8;
  NoallocTabArgs t;
  t.scratch = scratch;
  for (uint32_t first = 0; first < n; first += kNoallocTabChunk) {
    t.first = first;
    t.count = std::min(kNoallocTabChunk, n - first);
    for (uint32_t j = 0; j < t.count; ++j) t.e[j] = sorted ? room[first + j] : entry(first + j);
    if (const int err = launch(t)) return err;
  }
  return 0;
}

}  // namespace mma

#endif  // MMA_NOALLOC_H_
