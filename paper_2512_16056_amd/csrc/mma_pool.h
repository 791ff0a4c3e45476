// How a pool launch (a paged-KV transfer carried by one kernel, its pool in this
// GPU's memory or on the host) splits its pieces over waves. Plain arithmetic, shared by the launch,
// the kernels and a CPU test that emulates every wave over it.
//
// Units of work are numbered in the order of their destinations, and the
// hardware starts workgroups in that order, so that at any time the chip writes
// a few compact regions: HBM takes that best. A fetch writes pieces all over the
// layer tensors, an offload whole slots of the pool; so the table is sorted by
// destination, a fetch goes piece-major (piece p of neighbouring blocks is
// adjacent in the layer tensor) and an offload block-major.
// Measured, kernel alone, read+write, 1 GiB and 8 GiB of payload:
//                             32 KiB pieces               2 KiB pieces
//   fetch / offload           6.17, 5.93 / 6.14, 6.00     5.98, 5.65 / 5.91, 5.87 TB/s
//   the same, table unsorted  5.3 / 5.65                  5.2 / 5.2
//   fetch block-major         5.4, 5.2                    4.9
//   2, 4, 32 KiB per wave     6.06, 6.07, 5.51 (fetch, 1 GiB)
//   each XCD its own eighth   5.92, 5.91 / 5.84, 5.78     5.44, 5.64 / 5.65, 5.72
// and a plain copy of the same bytes 5.9 to 6.0. A host pool is taken block-major
// in table order, which reads or writes whole slots of it in a row.
#ifndef MMA_POOL_H_
#define MMA_POOL_H_

#include <stdint.h>

#if defined(__HIPCC__)
#define MMA_POOL_HD __host__ __device__
#else
#define MMA_POOL_HD
#endif

namespace mma {

// Division by a number known at launch: the estimate by its reciprocal is exact
// or one short.
struct FastDiv {
  uint32_t d, mul;
};
MMA_POOL_HD inline FastDiv fast_div(uint32_t d) {
  return FastDiv{d, d > 1 ? static_cast<uint32_t>((1ull << 32) / d) : 0xffffffffu};
}
MMA_POOL_HD inline uint32_t div_by(const FastDiv& f, uint32_t n) {
  const uint32_t q = static_cast<uint32_t>((static_cast<uint64_t>(n) * f.mul) >> 32);
  return n - q * f.d >= f.d ? q + 1 : q;
}

// 16-byte units one wave moves with one load per lane.
constexpr uint32_t kPoolRowUnits = 64;

// The pieces of a launch: number q is piece q / div of table entry q % div
// (by_piece: fetch, div = entries) or piece q % div of entry q / div (offload,
// div = pieces per block). n * ppb fits 32 bits.
struct PoolGeom {
  uint32_t by_piece;
  uint32_t total;    // pieces
  FastDiv div;
  // Rows of 64 units: a piece of 64 units or more takes rows.d of them, smaller
  // pieces share one, per_row each (rows.d = 1).
  uint32_t units;    // of a piece: 16 bytes each (x-packed values: lane tiles)
  FastDiv rows, piece_units;  // piece_units.d = units, where pieces share rows
  uint32_t per_row;
  uint64_t waves;
};

MMA_POOL_HD inline PoolGeom pool_geom(uint32_t n, uint32_t ppb, uint64_t units, uint32_t by_piece) {
  PoolGeom g;
  g.by_piece = by_piece;
  g.total = n * ppb;
  g.div = fast_div(by_piece ? n : ppb);
  g.units = static_cast<uint32_t>(units);
  const uint32_t u = g.units ? g.units : 1;
  const uint32_t rows = (u + kPoolRowUnits - 1) / kPoolRowUnits;
  g.rows = fast_div(rows);
  g.piece_units = fast_div(u < kPoolRowUnits ? u : kPoolRowUnits);
  g.per_row = u < kPoolRowUnits ? kPoolRowUnits / u : 1;
  g.waves = g.per_row > 1 ? (static_cast<uint64_t>(g.total) + g.per_row - 1) / g.per_row
                          : static_cast<uint64_t>(g.total) * rows;
  return g;
}

// The spans of one wave of a launch with fewer waves than spans: its own first,
// then every nw-th, or, with a claim counter, the next one nobody has taken (got:
// what the counter held). Over the link the waves' shares of it differ, and with
// fixed shares the slow ones leave it idle at the end: x-packed fetches 53.5 GB/s,
// with claims 57. There few spans go to as many workgroups as there are; in HBM a
// workgroup's are neighbours.
struct SpanWalk {
  uint64_t at, nw;
  uint32_t got;
};
MMA_POOL_HD inline SpanWalk span_walk(uint32_t wg, uint32_t grid, uint32_t wave, uint32_t waves_per_wg, bool link) {
  return SpanWalk{link ? static_cast<uint64_t>(wave) * grid + wg : static_cast<uint64_t>(wg) * waves_per_wg + wave,
                  static_cast<uint64_t>(grid) * waves_per_wg, 0};
}
MMA_POOL_HD inline void span_next(SpanWalk& s, bool claims, uint32_t got) { s.at = claims ? s.nw + got : s.at + s.nw; }

// Rows per span of a launch over the link, and of staged x-packed keys; spans of so
// many rows; x-packed keys' rows per span, whose spans come before the values', of one
// row each.
constexpr uint32_t kLinkRows = 8;
MMA_POOL_HD inline uint64_t span_count(uint64_t rows, uint32_t per) { return (rows + per - 1) / per; }
MMA_POOL_HD constexpr uint32_t xp_key_rows(bool link, bool stage) { return link || stage ? kLinkRows : 1; }

// Workgroups of a launch; most: over the link, else 0. A launch has fewer than 2^32
// threads; beyond that the waves go round again.
MMA_POOL_HD inline uint64_t pool_grid(uint64_t spans, uint32_t waves_per_wg, uint32_t most) {
  const uint64_t grid = (spans + waves_per_wg - 1) / waves_per_wg, limit = most ? most : 1u << 23;
  return grid < limit ? grid : limit;
}

// Above this many workgroups (64 MiB at 4 KiB each) counting them costs more than a
// second launch that writes the done tag: 1 GiB 371 / 354 us, 4 GiB 1498 / 1438.
constexpr uint64_t kPoolTagLaunch = 16384;

// Groups in which the workgroups of a launch count when they finish, at least 16
// to a group. A launch whose waves claim spans counts in one, whatever its grid:
// its claim counter stands where the first group's counter would. Its workgroups
// are few.
MMA_POOL_HD inline uint32_t pool_groups(uint32_t grid, bool claims, uint32_t most) {
  const uint32_t groups = grid / 16u < most ? grid / 16u : most;
  return claims || groups == 0 ? 1 : groups;
}


// What workgroup `wg` of `grid` does when it has finished: true for the one that
// finished last, with every counter back at 0 in memory. Counter 0 counts the
// groups (one group: its workgroups), 1 + i the workgroups of group i, or 1 the
// claims. c.add(i) adds 1 to counter i and returns what it held, c.zero(i) stores
// 0 in it, c.landed() waits until this wave's stores are in memory.
template <class Counters>
MMA_POOL_HD inline bool pool_last(uint32_t wg, uint32_t grid, bool claims, uint32_t most, Counters c) {
  const uint32_t groups = pool_groups(grid, claims, most);
  if (groups > 1) {
    const uint32_t i = wg % groups, members = (grid - i + groups - 1) / groups;
    if (c.add(1 + i) != members - 1) return false;
    c.zero(1 + i);
    c.landed();  // the count below lets the last workgroup, another wave, free this counter
  }
  if (c.add(0) != (groups > 1 ? groups : grid) - 1) return false;
  c.zero(0);
  if (claims) c.zero(1);
  c.landed();
  return true;
}

// A fetch without allocations has no slot of the engine and no counters of its own.
// Those that claim spans take 32 words in turn, 16 in each of two 128-byte lines, and
// the n-th of them sets the word of the (n + 16)-th, in the other line, to 0: it
// relies on nothing else that an earlier launch left behind, and counts no
// workgroups. So up to 16 calls that overlap, which is their callers' mistake, spoil
// neither each other's claims nor any later call's, and more of them the next 16 at
// most.
constexpr uint32_t kClaimAhead = 16, kClaimWords = 64, kClaimLone = 16;
MMA_POOL_HD inline uint32_t claim_word(uint32_t n) { return n / kClaimAhead % 2 * 32 + n % kClaimAhead; }
MMA_POOL_HD inline uint32_t claim_clears(uint32_t n) { return claim_word(n + kClaimAhead); }

// Table entry and piece of its block of piece number q.
struct PoolPiece {
  uint32_t entry, p;
};
MMA_POOL_HD inline PoolPiece pool_piece(const PoolGeom& g, uint32_t q) {
  const uint32_t hi = div_by(g.div, q), lo = q - hi * g.div.d;
  return PoolPiece{g.by_piece ? lo : hi, g.by_piece ? hi : lo};
}

// What a lane of wave w moves: unit u of piece number q, if ok.
struct PoolUnit {
  uint32_t q, u;
  bool ok;
};
MMA_POOL_HD inline PoolUnit pool_unit(const PoolGeom& g, uint32_t w, uint32_t lane) {
  PoolUnit x;
  if (g.per_row > 1) {
    const uint32_t j = div_by(g.piece_units, lane);
    x.q = w * g.per_row + j;
    x.u = lane - j * g.units;
    x.ok = j < g.per_row && x.q < g.total;
  } else {
    x.q = div_by(g.rows, w);
    x.u = (w - x.q * g.rows.d) * kPoolRowUnits + lane;
    x.ok = x.u < g.units;
  }
  return x;
}

// Head-major blocks: a piece is X x Y rows of C units, stored [X][Y][C] on the
// side whose order the lanes follow and [Y][X][C] on the other one. In HBM they
// follow the destination (fetch: X = heads, Y = tokens; offload: the reverse),
// over the link the host piece (X = tokens, Y = heads), so that PCIe requests
// stay whole: a fetch that followed its destination read 160-byte rows at
// 35-43 GB/s. The other side's unit for unit u.
struct HndMap {
  uint32_t X;
  FastDiv Y, C;
};
MMA_POOL_HD inline HndMap hnd_map(uint32_t X, uint32_t Y, uint32_t C) { return HndMap{X, fast_div(Y), fast_div(C)}; }
MMA_POOL_HD inline uint32_t hnd_other(const HndMap& m, uint32_t u) {
  const uint32_t row = div_by(m.C, u), x = div_by(m.Y, row);
  return ((row - x * m.Y.d) * m.X + x) * m.C.d + (u - row * m.C.d);
}

// Over the link with few workgroups each wave needs more in flight than the rows of a
// span, 8 KiB: pieces of 16 KiB and more, as they are on the host, go by wave_copy, up
// to kLinkFewSpan at a time. 64 MiB in 32 KiB pieces, 3 and 6 workgroups: by rows 2634
// and 1710 us, so 1613 and 1192; 16 KiB pieces 1785 and 1194. And x-packed claims are
// of as much: 64 MiB in 8 KiB pieces, 2 and 3 workgroups, 4973 / 4521 and 3223 / 2866.
constexpr uint32_t kLinkFewWgs = 12, kLinkFewSpan = 64 * 1024;
MMA_POOL_HD inline bool link_few(uint32_t wgs) { return wgs && wgs < kLinkFewWgs; }
MMA_POOL_HD inline bool link_long_spans(uint32_t wgs, uint64_t piece) { return link_few(wgs) && piece >= 16 * 1024; }

// x-packed blocks. A piece is B tokens of HC 16-byte units (x = 16 / element bytes
// elements each) on the host, [B][HC]. A key block holds the same units as [HC][B],
// a value block rows of B elements per dimension, [HC * x][B]: so a key lane moves
// one unit, and a value lane x units of x tokens by x dimensions, transposed in its
// registers. Keys and values have a geometry each, over the layers' pieces (ppb =
// layers).
// Unit v of a key piece: 8 x 8 units per wave where both sides divide, for runs of
// 128 bytes on either side; else the block's order.
// Lane tile v of a value piece: the block's order, runs of B elements there and of
// 64 / (B / x) units on the host.
struct XpMap {
  uint32_t B, HC;
  FastDiv tokens, groups, squares;  // by B, by B / x, by B / 8
  uint32_t square;                  // 1: 8 x 8
};
MMA_POOL_HD inline XpMap xp_map(uint32_t B, uint32_t HC, uint32_t x) {
  return XpMap{B, HC, fast_div(B), fast_div(B / x), fast_div(B >= 8 ? B / 8 : 1), B % 8 == 0 && HC % 8 == 0 ? 1u : 0u};
}
struct XpAt {
  uint32_t hc, t;  // key: unit and token; value: unit and token group
};
MMA_POOL_HD inline XpAt xp_key(const XpMap& m, uint32_t v) {
  if (m.square) {
    const uint32_t blk = v >> 6, in = v & 63, h = div_by(m.squares, blk), t = blk - h * m.squares.d;
    return XpAt{h * 8 + (in >> 3), t * 8 + (in & 7)};
  }
  const uint32_t hc = div_by(m.tokens, v);
  return XpAt{hc, v - hc * m.B};
}
MMA_POOL_HD inline XpAt xp_val(const XpMap& m, uint32_t v) {
  const uint32_t hc = div_by(m.groups, v);
  return XpAt{hc, v - hc * m.groups.d};
}
// Byte offsets in the host piece and in the block.
MMA_POOL_HD inline uint32_t xp_host(const XpMap& m, uint32_t hc, uint32_t t) { return (t * m.HC + hc) * 16; }
MMA_POOL_HD inline uint32_t xp_key_block(const XpMap& m, uint32_t hc, uint32_t t) { return (hc * m.B + t) * 16; }
MMA_POOL_HD inline uint32_t xp_val_block(const XpMap& m, uint32_t dim, uint32_t group) {
  return (dim * m.groups.d + group) * 16;
}

// A row of 64 value tiles covers 64 * x units of the block in a row, 8 KiB of 2-byte
// elements, where B / x divides 64 and pieces have rows of their own. It can then
// go through a tile in LDS, so that every access to the block is 1 KiB in a row:
// unit u of the row is kept at xp_stage_at(u), and xp_stage_unit is the unit that
// lane `lane` holds in its register i (of the block's order). The exchange of units
// within a run of x dimensions spreads the lanes' accesses over the banks.
MMA_POOL_HD inline bool xp_stages(uint64_t piece, uint32_t B, uint32_t elem) {
  const uint32_t x = 16 / elem, groups = B / x;
  return piece / 16 / x >= kPoolRowUnits && groups <= kPoolRowUnits && (groups & (groups - 1)) == 0;
}
template <uint32_t X>
MMA_POOL_HD inline uint32_t xp_stage_unit(const XpMap& m, uint32_t lane, uint32_t i) {
  return (div_by(m.groups, lane) * X + i) * m.groups.d + (lane & (m.groups.d - 1));
}
template <uint32_t X>
MMA_POOL_HD inline uint32_t xp_stage_at(const XpMap& m, uint32_t u) {
  return u ^ (div_by(m.groups, u) / X % X * m.groups.d);
}

}  // namespace mma

#endif  // MMA_POOL_H_
