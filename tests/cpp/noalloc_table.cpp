// The block table of a fetch without allocations (paper_2512_16056_amd/csrc/mma_noalloc.h) with
// launches made here: what reaches the launch, in its arguments or in the scratch array; a launch that
// fails; and a call whose launch waits while other threads make theirs. Built and run by
// tests/test_noalloc_table.py.
#include <cstdio>
#include <future>
#include <numeric>
#include <random>

#include "mma_noalloc.h"

using namespace mma;

static int failures = 0;
#define CHECK(c, ...)             \
  do {                            \
    if (!(c)) {                   \
      std::printf(__VA_ARGS__);   \
      std::printf("\n");          \
      ++failures;                 \
    }                             \
  } while (0)

struct Tables {
  std::vector<int32_t> hs, gb;
  explicit Tables(uint32_t n) : hs(n), gb(n) {
    std::iota(gb.begin(), gb.end(), 5);
    std::mt19937 rng(n);
    std::shuffle(gb.begin(), gb.end(), rng);
    for (uint32_t i = 0; i < n; ++i) hs[i] = static_cast<int32_t>(rng() % (2 * n));
  }
  std::vector<uint64_t> want(bool sorted) const {
    std::vector<uint64_t> w;
    for (size_t i = 0; i < hs.size(); ++i)
      w.push_back(static_cast<uint64_t>(hs[i]) | static_cast<uint64_t>(gb[i]) << 32);
    if (sorted) std::sort(w.begin(), w.end(), [](uint64_t a, uint64_t b) { return a >> 32 < b >> 32; });
    return w;
  }
};

static void tables(uint32_t layers) {
  std::vector<uint64_t> scratch(kNoallocScratchBytes / 8);
  for (uint32_t n : {1u, 63u, 64u, kPoolWords - layers, kPoolWords - layers + 1, 896u, 1000u, kNoallocMaxBlocks, 500u})
    for (bool sorted : {false, true}) {
      const Tables t(n);
      std::fill(scratch.begin(), scratch.end(), ~0ull);
      std::unique_ptr<PoolArgs> a(new PoolArgs());
      a->layers = a->words = layers;
      uint32_t launches = 0;
      const int rc = noalloc_table(*a, scratch.data(), t.hs.data(), t.gb.data(), n, sorted, [&](const NoallocTabArgs& l) {
        ++launches;
        CHECK(l.count <= kNoallocTabChunk && l.first + l.count <= n, "chunk %u + %u of %u", l.first, l.count, n);
        for (uint32_t j = 0; j < l.count; ++j) l.scratch[kNoallocTabOffset / 8 + l.first + j] = l.e[j];
        return 0;
      });
      const bool fits = layers + n <= kPoolWords;
      const uint64_t* got = fits ? a->w + layers : a->tab;
      CHECK(rc == 0 && launches == (fits ? 0 : (n + kNoallocTabChunk - 1) / kNoallocTabChunk), "%u launches for %u blocks",
            launches, n);
      CHECK(a->words == (fits ? layers + n : layers) && fits == (a->tab == nullptr), "words %u", a->words);
      const auto want = t.want(sorted);
      CHECK(std::equal(want.begin(), want.end(), got), "table of %u blocks, sorted %d, differs", n, sorted);
    }
}

static void failed_launch() {
  const Tables t(2000);
  std::unique_ptr<PoolArgs> a(new PoolArgs());
  std::vector<uint64_t> scratch(kNoallocScratchBytes / 8);
  uint32_t launches = 0;
  const int rc = noalloc_table(*a, scratch.data(), t.hs.data(), t.gb.data(), 2000, true,
                               [&](const NoallocTabArgs&) { return ++launches == 2 ? 719 : 0; });
  CHECK(rc == 719 && launches == 2, "a failed launch: %d after %u", rc, launches);
}

static void a_launch_that_waits() {
  const Tables t(1000);
  for (bool sorted : {false, true}) {
    std::promise<void> waiting, gate;
    std::shared_future<void> open = gate.get_future().share();
    std::vector<uint64_t> s1(kNoallocScratchBytes / 8), s2(s1.size());
    std::thread first([&] {
      std::unique_ptr<PoolArgs> a(new PoolArgs());
      bool told = false;
      noalloc_table(*a, s1.data(), t.hs.data(), t.gb.data(), 1000, sorted, [&](const NoallocTabArgs&) {
        if (!told) waiting.set_value();
        told = true;
        open.wait();
        return 0;
      });
    });
    waiting.get_future().wait();
    std::promise<void> over;
    std::future<void> done = over.get_future();
    std::thread second([&] {
      for (uint32_t n : {10u, 1000u}) {
        std::unique_ptr<PoolArgs> a(new PoolArgs());
        noalloc_table(*a, s2.data(), t.hs.data(), t.gb.data(), n, sorted, [](const NoallocTabArgs&) { return 0; });
      }
      over.set_value();
    });
    CHECK(done.wait_for(std::chrono::seconds(5)) == std::future_status::ready,
          "a call waits for another one's launch (sorted %d)", sorted);
    gate.set_value();
    first.join();
    second.join();
  }
}

int main() {
  for (uint32_t layers : {1u, 32u, kMaxLayers}) tables(layers);
  failed_launch();
  a_launch_that_waits();
  if (!failures) std::printf("ALL OK\n");
  return failures ? 1 : 0;
}
