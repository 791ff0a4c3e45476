// CPU emulation of a pool launch, in HBM (link = 0) or over the link, over the kernel's own index maps
// (paper_2512_16056_amd/csrc/mma_pool.h): every wave, row and lane,
// in the piece layout (hnd = 0) or the head-major one. Every access is checked
// against its buffer, and every byte of the destination pieces must be written
// exactly once. Built by tests/test_pool_index.py and compared there with the
// oracle.
#include <cstdint>
#include <cstring>
#include <vector>

#include "mma_pool.h"

using namespace mma;

// pool: slots of ppb pieces; cache: [layers][2][nb][piece]; tab: slot | block << 32.
extern "C" int emu_pool(uint8_t* pool, uint64_t pool_bytes, uint8_t* cache, uint64_t cache_bytes, const uint64_t* tab,
                        uint32_t n, uint32_t ppb, uint64_t piece, uint32_t nb, int to_paged, int hnd, int link,
                        uint32_t B, uint32_t H, uint32_t R) {
  const PoolGeom g = pool_geom(n, ppb, piece, to_paged && !link ? 1 : 0);
  const HndMap m = to_paged && !link ? hnd_map(H, B, R / 16) : hnd_map(B, H, R / 16);
  std::vector<uint8_t> wrote(to_paged ? cache_bytes : pool_bytes, 0);
  const uint8_t* src = to_paged ? pool : cache;
  uint8_t* dst = to_paged ? cache : pool;
  const uint64_t src_bytes = to_paged ? pool_bytes : cache_bytes, dst_bytes = to_paged ? cache_bytes : pool_bytes;
  for (uint64_t w = 0; w < g.waves; ++w) {
    for (uint32_t lane = 0; lane < 64; ++lane) {
      const PoolUnit x = pool_unit(g, static_cast<uint32_t>(w), lane);
      if (!x.ok) continue;
      if (x.q >= g.total || x.u >= piece / 16) return 1;
      const PoolPiece pp = pool_piece(g, x.q);
      if (pp.entry >= n || pp.p >= ppb) return 2;
      const uint64_t e = tab[pp.entry];
      const uint64_t in_pool = (e & 0xffffffffull) * ppb * piece + pp.p * piece;
      const uint64_t in_cache = pp.p * nb * piece + (e >> 32) * piece;
      // the lanes follow the destination, over the link the pool
      const uint64_t other = (hnd ? hnd_other(m, x.u) : x.u) * 16ull, own = x.u * 16ull;
      const bool own_src = link && to_paged;
      const uint64_t from = (to_paged ? in_pool : in_cache) + (own_src ? own : other);
      const uint64_t to = (to_paged ? in_cache : in_pool) + (own_src ? other : own);
      if (from + 16 > src_bytes || to + 16 > dst_bytes) return 3;
      std::memcpy(dst + to, src + from, 16);
      for (uint32_t i = 0; i < 16; ++i)
        if (wrote[to + i]++) return 4;
    }
  }
  uint64_t total = 0;
  for (uint8_t v : wrote) total += v;
  return total == static_cast<uint64_t>(n) * ppb * piece ? 0 : 5;
}

// div_by against the division itself: 0, or a dividend + 1 that differs.
extern "C" uint64_t emu_div(uint32_t d, uint32_t first, uint32_t count) {
  const FastDiv f = fast_div(d);
  for (uint32_t i = 0; i < count; ++i)
    if (div_by(f, first + i) != (first + i) / d) return first + i + 1ull;
  return 0;
}
