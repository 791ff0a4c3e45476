// CPU emulation of a pool launch, in HBM (link = 0) or over the link by at most `link` workgroups, over
// the kernel's own walk and index maps (paper_2512_16056_amd/csrc/mma_pool.h): every wave, span, row and lane,
// in the piece layout (hnd = 0) or the head-major one. Every access is checked
// against its buffer, and every byte of the destination pieces must be written
// exactly once. Built by tests/test_pool_index.py and compared there with the
// oracle.
#include <cstdint>
#include <cstring>
#include <random>
#include <vector>

#include "mma_pool.h"

using namespace mma;

// The spans that the waves of a launch take, in the order they take them: the waves run in turn, one
// span each, with the claims (if any) on one counter.
static std::vector<uint64_t> walk(uint64_t spans, uint32_t wgs, bool claims) {
  const uint32_t waves = 4, grid = static_cast<uint32_t>(pool_grid(spans, waves, wgs));
  std::vector<SpanWalk> s;
  for (uint32_t g = 0; g < grid; ++g)
    for (uint32_t w = 0; w < waves; ++w) s.push_back(span_walk(g, grid, w, waves, wgs != 0));
  std::vector<uint64_t> taken;
  uint32_t counter = 0;
  for (bool any = true; any;) {
    any = false;
    for (SpanWalk& x : s)
      if (x.at < spans) {
        taken.push_back(x.at);
        span_next(x, claims, claims ? counter++ : 0);
        any = true;
      }
  }
  return taken;
}

// pool: slots of ppb pieces; cache: [layers][2][nb][piece]; tab: slot | block << 32.
extern "C" int emu_pool(uint8_t* pool, uint64_t pool_bytes, uint8_t* cache, uint64_t cache_bytes, const uint64_t* tab,
                        uint32_t n, uint32_t ppb, uint64_t piece, uint32_t nb, int to_paged, int hnd, int link,
                        int claims, uint32_t B, uint32_t H, uint32_t R) {
  const PoolGeom g = pool_geom(n, ppb, piece >> 4, to_paged && !link ? 1 : 0);
  const HndMap m = to_paged && !link ? hnd_map(H, B, R / 16) : hnd_map(B, H, R / 16);
  std::vector<uint8_t> wrote(to_paged ? cache_bytes : pool_bytes, 0);
  const uint8_t* src = to_paged ? pool : cache;
  uint8_t* dst = to_paged ? cache : pool;
  const uint64_t src_bytes = to_paged ? pool_bytes : cache_bytes, dst_bytes = to_paged ? cache_bytes : pool_bytes;
  const uint32_t per = link ? kLinkRows : 1;
  std::vector<uint64_t> rows;  // link: workgroups at most
  for (uint64_t s : walk(span_count(g.waves, per), static_cast<uint32_t>(link), claims != 0))
    for (uint64_t w = s * per; w < (s + 1) * per && w < g.waves; ++w) rows.push_back(w);
  for (uint64_t w : rows) {
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

// The highest counter (kPoolCtrStride words each) that the workgroups of a launch count on.
extern "C" uint32_t emu_last_counter(uint32_t grid, int claims, uint32_t most) {
  const uint32_t groups = pool_groups(grid, claims != 0, most);
  return groups > 1 ? groups : 0;
}

extern "C" int emu_long_spans(uint32_t wgs, uint64_t piece) { return link_long_spans(wgs, piece) ? 1 : 0; }

// Counters whose stores of 0 stay with the workgroup that made them until it waits (or, in the
// end, until it is over).
struct EmuCounters {
  std::vector<uint32_t>* mem;
  std::vector<uint32_t>* pending;  // of this workgroup
  uint32_t add(uint32_t i) const { return (*mem)[i]++; }
  void zero(uint32_t i) const { pending->push_back(i); }
  void landed() const {
    for (uint32_t i : *pending) (*mem)[i] = 0;
    pending->clear();
  }
};

// The workgroups of a launch finish in the order of `order`. 0 if the last one alone is told so,
// and at that moment no counter is short of its 0: the done tag written then frees them for
// another launch.
extern "C" int emu_finish(const uint32_t* order, uint32_t grid, int claims, uint32_t most) {
  std::vector<uint32_t> mem(1 + most, 0);
  if (claims) mem[1] = 12345;  // what the claims left
  std::vector<std::vector<uint32_t>> pending(grid);
  for (uint32_t k = 0; k < grid; ++k) {
    const bool last = pool_last(order[k], grid, claims != 0, most, EmuCounters{&mem, &pending[k]});
    if (last != (k == grid - 1)) return 1;
  }
  for (const auto& p : pending)
    if (!p.empty()) return 2;
  for (uint32_t v : mem)
    if (v) return 3;
  return 0;
}

// Launches of fetches without allocations that claim `spans` spans each, after `before` of them:
// `overlap` at once, their steps interleaved at random, then 40 one after another. 0 if every
// launch takes every span exactly once; else its number + 1.
extern "C" int emu_noalloc_claims(uint32_t before, uint32_t overlap, uint32_t waves, uint32_t spans, uint32_t seed) {
  std::vector<uint32_t> words(kClaimWords, 0);
  std::mt19937 rng(seed);
  struct Launch {
    uint32_t claim, clear;
    std::vector<uint64_t> at;       // of each wave
    std::vector<uint8_t> taken;
    bool cleared = false, once = true;
  };
  uint32_t n = 0;
  const auto run = [&](uint32_t count) {
    std::vector<Launch> ls(count);
    for (Launch& l : ls) {
      l.claim = claim_word(n);
      l.clear = claim_clears(n++);
      for (uint32_t w = 0; w < waves; ++w) l.at.push_back(w);
      l.taken.assign(spans, 0);
    }
    std::vector<std::pair<uint32_t, uint32_t>> steps;  // launch, wave (`waves`: its clearing)
    for (uint32_t i = 0; i < count; ++i)
      for (uint32_t w = 0; w <= waves; ++w) steps.emplace_back(i, w);
    while (!steps.empty()) {
      const size_t k = rng() % steps.size();
      Launch& l = ls[steps[k].first];
      const uint32_t w = steps[k].second;
      bool over = true;
      if (w == waves) {
        words[l.clear] = 0;
      } else if (l.at[w] < spans) {
        l.once &= !l.taken[l.at[w]]++;
        l.at[w] = waves + words[l.claim]++;
        over = false;
      }
      if (over) {
        steps[k] = steps.back();
        steps.pop_back();
      }
    }
    for (uint32_t i = 0; i < count; ++i) {
      for (uint8_t t : ls[i].taken) ls[i].once &= t == 1;
      if (!ls[i].once) return static_cast<int>(n - count + i + 1);
    }
    return 0;
  };
  for (uint32_t i = 0; i < before; ++i)
    if (const int rc = run(1)) return rc;
  if (const int rc = run(overlap)) return rc;
  for (uint32_t i = 0; i < 40; ++i)
    if (const int rc = run(1)) return rc;
  return 0;
}

// The tile of a staged row: unit and place of every lane's register i. Bijective places, and the
// same unit of the block as the lane would write by itself.
template <uint32_t X>
static int stage_row(const XpMap& m, const PoolGeom& g, uint64_t w) {
  bool place[64 * X] = {}, unit[64 * X] = {};
  const uint32_t first = pool_unit(g, static_cast<uint32_t>(w), 0).u;
  const uint32_t n = (g.units - first < 64 ? g.units - first : 64) * X;
  for (uint32_t u = 0; u < 64 * X; ++u) {
    const uint32_t at = xp_stage_at<X>(m, u);
    if (at >= 64 * X || place[at]) return 10;
    place[at] = true;
  }
  for (uint32_t lane = 0; lane < 64; ++lane) {
    const PoolUnit x = pool_unit(g, static_cast<uint32_t>(w), lane);
    if (!x.ok) continue;
    const XpAt a = xp_val(m, x.u);
    for (uint32_t i = 0; i < X; ++i) {
      const uint32_t u = xp_stage_unit<X>(m, lane, i);
      if (u >= n || unit[u]) return 11;
      unit[u] = true;
      if ((first * X + u) * 16 != xp_val_block(m, a.hc * X + i, a.t)) return 12;
    }
  }
  for (uint32_t u = 0; u < n; ++u)
    if (!unit[u]) return 13;
  return 0;
}

// x-packed blocks: key lanes move one unit, value lanes X units transposed, over
// the same maps. E: element bytes; HC: 16-byte units per token.
extern "C" int emu_pool_xp(uint8_t* pool, uint64_t pool_bytes, uint8_t* cache, uint64_t cache_bytes,
                           const uint64_t* tab, uint32_t n, uint32_t layers, uint64_t piece, uint32_t nb, int to_paged,
                           int link, int claims, uint32_t B, uint32_t HC, uint32_t E) {
  const uint32_t X = 16 / E, ppb = 2 * layers, by_piece = to_paged && !link ? 1 : 0;
  const XpMap m = xp_map(B, HC, X);
  const PoolGeom geom[2] = {pool_geom(n, layers, static_cast<uint64_t>(HC) * B, by_piece),
                            pool_geom(n, layers, static_cast<uint64_t>(HC) * (B / X), by_piece)};
  std::vector<uint8_t> wrote(to_paged ? cache_bytes : pool_bytes, 0);
  const uint8_t* src = to_paged ? pool : cache;
  uint8_t* dst = to_paged ? cache : pool;
  const uint64_t src_bytes = to_paged ? pool_bytes : cache_bytes, dst_bytes = to_paged ? cache_bytes : pool_bytes;
  if (!link && xp_stages(piece, B, E)) {
    for (uint64_t w = 0; w < geom[1].waves; ++w) {
      const int rc = X == 16  ? stage_row<16>(m, geom[1], w)
                     : X == 8 ? stage_row<8>(m, geom[1], w)
                     : X == 4 ? stage_row<4>(m, geom[1], w)
                              : stage_row<2>(m, geom[1], w);
      if (rc) return rc;
    }
  }
  // keys in spans of rows, then a row of values each
  const uint32_t per = xp_key_rows(link != 0, !link && xp_stages(piece, B, E));
  const uint64_t keys = span_count(geom[0].waves, per);
  std::vector<uint64_t> rows[2];
  for (uint64_t s : walk(keys + geom[1].waves, static_cast<uint32_t>(link), claims != 0)) {
    if (s >= keys) rows[1].push_back(s - keys);
    for (uint64_t w = s * per; s < keys && w < (s + 1) * per && w < geom[0].waves; ++w) rows[0].push_back(w);
  }
  for (uint32_t kind = 0; kind < 2; ++kind) {
    const PoolGeom& g = geom[kind];
    for (uint64_t w : rows[kind])
      for (uint32_t lane = 0; lane < 64; ++lane) {
        const PoolUnit x = pool_unit(g, static_cast<uint32_t>(w), lane);
        if (!x.ok) continue;
        if (x.q >= g.total || x.u >= g.units) return 1;
        const PoolPiece pp = pool_piece(g, x.q);
        if (pp.entry >= n || pp.p >= layers) return 2;
        const uint64_t e = tab[pp.entry], p = 2 * pp.p + kind;
        const uint64_t in_pool = (e & 0xffffffffull) * ppb * piece + p * piece;
        const uint64_t in_cache = p * nb * piece + (e >> 32) * piece;
        const uint64_t from = to_paged ? in_pool : in_cache, to = to_paged ? in_cache : in_pool;
        uint8_t in[16 * 16], out[16 * 16];
        uint64_t so[16], to_off[16];
        const uint32_t count = kind ? X : 1;
        for (uint32_t i = 0; i < count; ++i) {
          uint64_t host, blk;
          if (kind) {
            const XpAt a = xp_val(m, x.u);
            host = xp_host(m, a.hc, a.t * X + i);
            blk = xp_val_block(m, a.hc * X + i, a.t);
          } else {
            const XpAt a = xp_key(m, x.u);
            host = xp_host(m, a.hc, a.t);
            blk = xp_key_block(m, a.hc, a.t);
          }
          if (host + 16 > piece || blk + 16 > piece) return 3;
          so[i] = from + (to_paged ? host : blk);
          to_off[i] = to + (to_paged ? blk : host);
          if (so[i] + 16 > src_bytes || to_off[i] + 16 > dst_bytes) return 4;
          std::memcpy(in + 16 * i, src + so[i], 16);
        }
        if (kind) {
          for (uint32_t j = 0; j < X; ++j)
            for (uint32_t i = 0; i < X; ++i) std::memcpy(out + 16 * j + i * E, in + 16 * i + j * E, E);
        } else {
          std::memcpy(out, in, 16);
        }
        for (uint32_t j = 0; j < count; ++j) {
          std::memcpy(dst + to_off[j], out + 16 * j, 16);
          for (uint32_t i = 0; i < 16; ++i)
            if (wrote[to_off[j] + i]++) return 5;
        }
      }
  }
  uint64_t total = 0;
  for (uint8_t v : wrote) total += v;
  return total == static_cast<uint64_t>(n) * ppb * piece ? 0 : 6;
}
