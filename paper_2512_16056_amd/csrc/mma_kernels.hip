// Device side of the multipath copy path for gfx950 (MI355X).
//
// mma_transfer_kernel is the per-transfer "dummy task" (Section 3.3, Sync
// Engine; Section 4, Spin Kernel) enqueued on the caller's stream in place of
// the copy. Its waves do three things:
//   1. the first wave to run publishes `started` -- the stream -> engine start
//      signal (the paper uses a host callback for this direction);
//   2. every wave is a worker of the CU path (Section 3.4: one outstanding
//      queue per path): it claims ring entries with a device-memory atomic and
//      moves them with wide zero-copy loads/stores across PCIe, or between the
//      paged KV layout and SDMA staging buffers in HBM; each wave signals its
//      own completions (wavefront-level completion);
//   3. the last wave to finish claiming holds the stream until the engine
//      reports that every micro-task of every path has landed (the spin wait
//      of Section 4), with a bounded, progress-re-armed watchdog, then exits
//      and releases downstream stream work.
// Under device control the whole CU share is in the ring before the launch
// (a ticket past it ends a wave's claims) and the last wave waits for the copy
// engines' own completion signal instead of the engine's word: no host thread
// takes part once the kernel runs. mma_transfer_xpacked_kernel<E> is the same
// kernel for the x-packed GPU block layout (an LDS transform per piece),
// mma_transfer_hnd_kernel for the head-major one (a row permutation), and
// mma_whole_kernel<N> a self-contained launch whose N entries travel in its
// arguments.
//
// Every host-memory poll is a PCIe read that competes with the payload for the
// link, so polls are few: one load instruction both checks and fetches a ring
// entry, an idle wave backs off exponentially, and the close/heartbeat words
// are read only every few polls.
//
// mma_digest_kernel is the dependent HBM-bound check kernel of the
// mixed-contention workload.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "mma_proto.h"
#include "mma_xpacked.h"

namespace mma {
namespace {

// Global-address-space views: global_load/global_store instead of flat ones
// (no LDS-counter waits on the copy path).
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) u32x4 gu4;

__device__ __forceinline__ uint64_t ld_sys(const uint64_t* p) {
  return __hip_atomic_load(const_cast<uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ void st_sys(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__device__ __forceinline__ uint64_t lane_u64(uint64_t v, int lane) {
  const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(v), lane);
  const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(v >> 32), lane);
  return (static_cast<uint64_t>(hi) << 32) | lo;
}

__device__ __forceinline__ void backoff(uint32_t n) {
  for (uint32_t k = 0; k < n; ++k) __builtin_amdgcn_s_sleep(8);  // ~512 cycles each
}

// One batch = 16 loads of 16 B per lane = 16 KiB per wave.
constexpr uint64_t kBatch = 16 * kWave;  // in 16-byte units

#define MMA_LOAD16(V, base)                                                                                \
  V##0 = s[(base) + 0 * kWave]; V##1 = s[(base) + 1 * kWave]; V##2 = s[(base) + 2 * kWave];                \
  V##3 = s[(base) + 3 * kWave]; V##4 = s[(base) + 4 * kWave]; V##5 = s[(base) + 5 * kWave];                \
  V##6 = s[(base) + 6 * kWave]; V##7 = s[(base) + 7 * kWave]; V##8 = s[(base) + 8 * kWave];                \
  V##9 = s[(base) + 9 * kWave]; V##10 = s[(base) + 10 * kWave]; V##11 = s[(base) + 11 * kWave];            \
  V##12 = s[(base) + 12 * kWave]; V##13 = s[(base) + 13 * kWave]; V##14 = s[(base) + 14 * kWave];          \
  V##15 = s[(base) + 15 * kWave];
#define MMA_STORE16(V, base)                                                                               \
  d[(base) + 0 * kWave] = V##0; d[(base) + 1 * kWave] = V##1; d[(base) + 2 * kWave] = V##2;                \
  d[(base) + 3 * kWave] = V##3; d[(base) + 4 * kWave] = V##4; d[(base) + 5 * kWave] = V##5;                \
  d[(base) + 6 * kWave] = V##6; d[(base) + 7 * kWave] = V##7; d[(base) + 8 * kWave] = V##8;                \
  d[(base) + 9 * kWave] = V##9; d[(base) + 10 * kWave] = V##10; d[(base) + 11 * kWave] = V##11;            \
  d[(base) + 12 * kWave] = V##12; d[(base) + 13 * kWave] = V##13; d[(base) + 14 * kWave] = V##14;          \
  d[(base) + 15 * kWave] = V##15;

// n16 16-byte units s[0, n16) -> d[0, n16), both aligned. Consecutive lanes
// move consecutive units, so each load instruction covers one contiguous 1 KiB
// span. Two register batches ping-pong: the loads of the next batch are issued
// before the current batch is stored, so a wave keeps up to 32 KiB of reads in
// flight.
__device__ __forceinline__ void aligned_units(const gu4* __restrict__ s0, gu4* __restrict__ d0, uint64_t n16,
                                              uint32_t lane) {
  const gu4* s = s0 + lane;  // this lane's unit
  gu4* d = d0 + lane;
  const uint64_t nb = n16 / kBatch;  // full batches (wave-uniform)
  if (nb > 0) {
    u32x4 a0, a1, a2, a3, a4, a5, a6, a7, a8, a9, a10, a11, a12, a13, a14, a15;
    u32x4 b0, b1, b2, b3, b4, b5, b6, b7, b8, b9, b10, b11, b12, b13, b14, b15;
    MMA_LOAD16(a, 0)
    uint64_t k = 0;  // batch held in registers `a` at the top of the loop
    for (;;) {
      if (k + 1 >= nb) {
        MMA_STORE16(a, k * kBatch)
        break;
      }
      MMA_LOAD16(b, (k + 1) * kBatch)
      __builtin_amdgcn_sched_barrier(0);
      MMA_STORE16(a, k * kBatch)
      ++k;
      if (k + 1 >= nb) {
        MMA_STORE16(b, k * kBatch)
        break;
      }
      MMA_LOAD16(a, (k + 1) * kBatch)
      __builtin_amdgcn_sched_barrier(0);
      MMA_STORE16(b, k * kBatch)
      ++k;
    }
  }
  // Remainder (< one batch): one batch, all loads issued before the first
  // store, so a short copy costs one round trip instead of one per 1 KiB. The
  // loads are unconditional -- a lane past the end re-reads the last unit -- and
  // only the stores are predicated: a predicated load makes the compiler wait
  // for it before the next one, one PCIe round trip each.
  const uint64_t r = nb * kBatch;
  if (r < n16) {
    const uint64_t left = n16 - r;  // units left for the whole wave, < kBatch
    u32x4 c0, c1, c2, c3, c4, c5, c6, c7, c8, c9, c10, c11, c12, c13, c14, c15;
#define MMA_PLD(k) c##k = s0[r + min(static_cast<uint64_t>((k) * kWave + lane), left - 1)];
#define MMA_PST(k) if ((k) * kWave + lane < left) d[r + (k) * kWave] = c##k;
    MMA_PLD(0) MMA_PLD(1) MMA_PLD(2) MMA_PLD(3) MMA_PLD(4) MMA_PLD(5) MMA_PLD(6) MMA_PLD(7)
    MMA_PLD(8) MMA_PLD(9) MMA_PLD(10) MMA_PLD(11) MMA_PLD(12) MMA_PLD(13) MMA_PLD(14) MMA_PLD(15)
    __builtin_amdgcn_sched_barrier(0);
    MMA_PST(0) MMA_PST(1) MMA_PST(2) MMA_PST(3) MMA_PST(4) MMA_PST(5) MMA_PST(6) MMA_PST(7)
    MMA_PST(8) MMA_PST(9) MMA_PST(10) MMA_PST(11) MMA_PST(12) MMA_PST(13) MMA_PST(14) MMA_PST(15)
#undef MMA_PLD
#undef MMA_PST
  }
}

// Bytes [4Q + r, 4Q + r + 16) of the 32 bytes lo|hi (little-endian), r < 4:
// v_alignbyte_b32 takes 4 bytes at a byte offset out of two adjacent words.
template <uint32_t Q>
__device__ __forceinline__ u32x4 funnel16(const u32x4& lo, const u32x4& hi, uint32_t r) {
  const uint32_t w[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  u32x4 o;
  o[0] = __builtin_amdgcn_alignbyte(w[Q + 1], w[Q], r);
  o[1] = __builtin_amdgcn_alignbyte(w[Q + 2], w[Q + 1], r);
  o[2] = __builtin_amdgcn_alignbyte(w[Q + 3], w[Q + 2], r);
  o[3] = __builtin_amdgcn_alignbyte(w[Q + 4], w[Q + 3], r);
  return o;
}

// One batch of a realigning copy: rows v[0..15] hold source units
// base + i * 64 + lane; `next` is unit base + kBatch, the same in every lane.
// A lane's unit k + 1 is its right neighbour's unit k (ds_bpermute); lane
// 63's is lane 0's of the next row (readlane), or `next` for the last row.
template <uint32_t Q>
__device__ __forceinline__ void realign_store(const u32x4 (&v)[16], const u32x4& next, gu4* __restrict__ d,
                                              uint64_t base, uint64_t n16, uint32_t r, uint32_t lane, int right) {
#pragma unroll
  for (uint32_t i = 0; i < 16; ++i) {
    u32x4 hi;
#pragma unroll
    for (uint32_t w = 0; w < 4; ++w) {
      const uint32_t nb = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(right, static_cast<int>(v[i][w])));
      const uint32_t l0 = i < 15 ? __builtin_amdgcn_readlane(v[i + 1][w], 0) : next[w];
      hi[w] = lane == kWave - 1 ? l0 : nb;
    }
    const uint64_t u = base + i * kWave + lane;
    if (u < n16) d[u] = funnel16<Q>(v[i], hi, r);
  }
}

// n16 aligned destination units d[0, n16) from a source that starts
// s = 4Q + r bytes (1 <= s <= 15) past the aligned unit sa[0]: unit k is bytes
// [s, s + 16) of the aligned source units k and k + 1. Every load and store is
// an aligned 16-byte unit; the shift happens in registers. Source units
// [0, n16] each hold at least one byte of the source range, and loads past
// the end are clamped to unit n16, so no load leaves the aligned units the
// range touches; stores are predicated.
// kDeep = false: one 16 KiB batch in flight per wave; a batch's `next` unit is
// one more load that every lane makes at the same address (one request).
// kDeep = true: batches ping-pong as in aligned_units -- the next batch's loads
// are issued before this one is stored, and its first unit is this batch's
// `next` -- for 32 KiB in flight per wave; the last batch's `next`, unit n16,
// is read once at the start. It needs 64 more VGPRs, which only the lean
// self-contained kernel has to spare.
template <uint32_t Q, bool kDeep>
__device__ void realign_units(const gu4* __restrict__ sa, gu4* __restrict__ d, uint64_t n16, uint32_t r,
                              uint32_t lane) {
  const int right = static_cast<int>(((lane + 1) & (kWave - 1)) << 2);  // ds_bpermute byte address
  auto load = [&](u32x4 (&v)[16], uint64_t base) {
#pragma unroll
    for (uint32_t i = 0; i < 16; ++i) v[i] = sa[min(base + i * kWave + lane, n16)];
  };
  if constexpr (!kDeep) {
    for (uint64_t base = 0; base < n16; base += kBatch) {
      u32x4 v[16];
      load(v, base);
      const u32x4 next = sa[min(base + kBatch, n16)];
      __builtin_amdgcn_sched_barrier(0);
      realign_store<Q>(v, next, d, base, n16, r, lane, right);
    }
  } else {
    const u32x4 last = sa[n16];
    auto first = [&](const u32x4& v0) {
      u32x4 x;
#pragma unroll
      for (uint32_t w = 0; w < 4; ++w) x[w] = __builtin_amdgcn_readlane(v0[w], 0);
      return x;
    };
    u32x4 a[16], b[16];
    load(a, 0);
    for (uint64_t base = 0;;) {
      if (base + kBatch >= n16) {
        realign_store<Q>(a, last, d, base, n16, r, lane, right);
        break;
      }
      load(b, base + kBatch);
      __builtin_amdgcn_sched_barrier(0);
      realign_store<Q>(a, first(b[0]), d, base, n16, r, lane, right);
      base += kBatch;
      if (base + kBatch >= n16) {
        realign_store<Q>(b, last, d, base, n16, r, lane, right);
        break;
      }
      load(a, base + kBatch);
      __builtin_amdgcn_sched_barrier(0);
      realign_store<Q>(b, first(a[0]), d, base, n16, r, lane, right);
      base += kBatch;
    }
  }
}

// Wave-cooperative copy of n bytes. A byte head brings the destination to a
// 16-byte boundary; the aligned middle moves in 16-byte units -- straight
// (aligned_units) when source and destination are equally aligned modulo 16,
// else realigned in registers (realign_units); a byte tail finishes. The head
// and tail bytes are read first, with unconditional clamped loads, and
// written last, so their round trips overlap the middle's instead of
// preceding it. kDeep: see realign_units.
template <bool kDeep = false>
__device__ __forceinline__ void wave_copy(const uint8_t* __restrict__ src, uint8_t* __restrict__ dst,
                                          uint64_t n, uint32_t lane) {
  const bool rel = ((reinterpret_cast<uintptr_t>(src) ^ reinterpret_cast<uintptr_t>(dst)) & 15u) != 0;
  uint64_t head = (16u - (reinterpret_cast<uintptr_t>(dst) & 15u)) & 15u;
  if (head > n) head = n;
  const uint64_t n16 = (n - head) >> 4, tail = (n - head) & 15u, tb = head + (n16 << 4);
  uint8_t hv = 0, tv = 0;
  if (head) hv = src[min(static_cast<uint64_t>(lane), head - 1)];
  if (tail) tv = src[tb + min(static_cast<uint64_t>(lane), tail - 1)];
  if (n16) {
    const uint8_t* s = src + head;
    gu4* d = (gu4*)(dst + head);
    if (!rel) {
      aligned_units((const gu4*)(s), d, n16, lane);
    } else {
      const uint32_t sh = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(s) & 15u);
      const gu4* sa = (const gu4*)(s - sh);
      switch (sh >> 2) {
        case 0: realign_units<0, kDeep>(sa, d, n16, sh & 3u, lane); break;
        case 1: realign_units<1, kDeep>(sa, d, n16, sh & 3u, lane); break;
        case 2: realign_units<2, kDeep>(sa, d, n16, sh & 3u, lane); break;
        default: realign_units<3, kDeep>(sa, d, n16, sh & 3u, lane); break;
      }
    }
  }
  if (lane < head) dst[lane] = hv;
  if (lane < tail) dst[tb + lane] = tv;
}

// ---------------------------------------------------------------- x-packed KV layout
// A paged-KV piece in the x-packed layout: key [H][R/16][B][16 bytes], value
// [H][D][B] elements, while the host keeps every piece token-major [B][H][R]
// (R = head_dim * elem bytes per token row of one head). Both transforms
// permute the piece at 16-byte (key) or element (value) granularity, so one
// side of a direct copy would be read or written in scattered 16-byte or
// smaller pieces -- across PCIe, requests that small waste most of each
// transaction. Each wave therefore stages a group of whole heads in its slice
// of LDS: it reads the group coalesced in the source's order, then writes it
// coalesced in the destination's order, gathering from LDS. Rows in LDS are
// padded by 16 bytes to spread the column reads over the banks.
typedef __attribute__((address_space(3))) uint8_t lds_u8;
typedef __attribute__((address_space(3))) u32x4 lu4;

// Make LDS writes of the wave visible to its other lanes (the wave-level
// barrier idiom: release, wave barrier, acquire).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 16-byte units [0, n) moved by one wave: map(u) gives the unit's source and
// destination offsets, get(source offset) reads it, put(destination offset, v)
// writes it. kUnits units per lane are read before the first is written; their
// offsets are computed once and kept in registers.
constexpr uint32_t kUnits = 8;
struct UnitOffs {
  uint32_t src, dst;
};
// Reads are unconditional (a lane past the end reads unit n - 1 again): a
// predicated read would make the compiler wait for it before issuing the next.
template <class Map, class Get, class Put>
__device__ __forceinline__ void wave_units(uint32_t n, uint32_t lane, Map map, Get get, Put put) {
  for (uint32_t base = 0; base < n; base += kUnits * kWave) {
    u32x4 v[kUnits];
    UnitOffs o[kUnits];
#pragma unroll
    for (uint32_t i = 0; i < kUnits; ++i) {
      o[i] = map(min(base + i * kWave + lane, n - 1));
      v[i] = get(o[i].src);
    }
#pragma unroll
    for (uint32_t i = 0; i < kUnits; ++i) {
      if (base + i * kWave + lane < n) put(o[i].dst, v[i]);
    }
  }
}

// 16 bytes made of 16 / E elements of E bytes, element j at p + j * stride (LDS).
template <uint32_t E>
__device__ __forceinline__ u32x4 gather16(const lds_u8* p, uint32_t stride) {
  u32x4 r;
  if constexpr (E == 1) {
#pragma unroll
    for (uint32_t w = 0; w < 4; ++w) {
      const lds_u8* q = p + 4 * w * stride;
      r[w] = static_cast<uint32_t>(q[0]) | (static_cast<uint32_t>(q[stride]) << 8) |
             (static_cast<uint32_t>(q[2 * stride]) << 16) | (static_cast<uint32_t>(q[3 * stride]) << 24);
    }
  } else if constexpr (E == 2) {
#pragma unroll
    for (uint32_t w = 0; w < 4; ++w) {
      const auto* q0 = reinterpret_cast<const __attribute__((address_space(3))) uint16_t*>(p + 2 * w * stride);
      const auto* q1 = reinterpret_cast<const __attribute__((address_space(3))) uint16_t*>(p + (2 * w + 1) * stride);
      r[w] = static_cast<uint32_t>(*q0) | (static_cast<uint32_t>(*q1) << 16);
    }
  } else if constexpr (E == 4) {
#pragma unroll
    for (uint32_t w = 0; w < 4; ++w) r[w] = *reinterpret_cast<const __attribute__((address_space(3))) uint32_t*>(p + w * stride);
  } else {
#pragma unroll
    for (uint32_t w = 0; w < 2; ++w) {
      const auto* q = reinterpret_cast<const __attribute__((address_space(3))) uint32_t*>(p + w * stride);
      r[2 * w] = q[0];
      r[2 * w + 1] = q[1];
    }
  }
  return r;
}

// Heads [first, end) of host (token-major) piece `src` -> x-packed block `dst`; k = 0
// key, 1 value.
template <uint32_t E>
__device__ void xpacked_to_block(const uint8_t* src, uint8_t* dst, uint32_t k, const XGeom& g, lds_u8* lds,
                                 uint32_t lane, uint32_t first, uint32_t end) {
  const uint32_t G = xp_to_heads(g);
  auto to_lds = [&](uint32_t o, u32x4 v) { *reinterpret_cast<lu4*>(lds + o) = v; };
  for (uint32_t h0 = first; h0 < end; h0 += G) {
    const uint32_t gh = xp_min(G, end - h0), rs = xp_to_row_stride(g, gh);
    wave_units(xp_to_load_count(g, gh), lane,
               [&](uint32_t u) {
                 UnitOffs o;
                 xp_to_load(g, h0, gh, u, &o.src, &o.dst);
                 return o;
               },
               [&](uint32_t o) -> u32x4 { return *(const gu4*)(src + o); }, to_lds);
    wave_sync();
    uint8_t* out = dst + h0 * g.B * g.R;  // heads are the block's outermost dimension
    auto to_out = [&](uint32_t o, u32x4 v) { *(gu4*)(out + o) = v; };
    if (k == 0)
      wave_units(xp_to_key_count(g, gh), lane, [&](uint32_t v) { return UnitOffs{xp_to_key_lds(g, gh, v), v * 16}; },
                 [&](uint32_t o) -> u32x4 { return *reinterpret_cast<const lu4*>(lds + o); }, to_out);
    else
      wave_units(xp_to_val_count(g, gh), lane, [&](uint32_t v) { return UnitOffs{xp_to_val_lds(g, gh, v), v * 16}; },
                 [&](uint32_t o) -> u32x4 { return gather16<E>(lds + o, rs); }, to_out);
    wave_sync();  // the tile is read before the next group overwrites it
  }
}

// Heads [first, end) of x-packed block `src` -> host (token-major) piece `dst`; k = 0
// key, 1 value.
template <uint32_t E>
__device__ void xpacked_from_block(const uint8_t* src, uint8_t* dst, uint32_t k, const XGeom& g, lds_u8* lds,
                                   uint32_t lane, uint32_t first, uint32_t end) {
  const uint32_t G = xp_from_heads(g, k), rs = xp_from_row_stride(g, k);
  auto to_lds = [&](uint32_t o, u32x4 v) { *reinterpret_cast<lu4*>(lds + o) = v; };
  auto to_dst = [&](uint32_t o, u32x4 v) { *(gu4*)(dst + o) = v; };
  for (uint32_t h0 = first; h0 < end; h0 += G) {
    const uint32_t gh = xp_min(G, end - h0);
    const uint8_t* in = src + h0 * g.B * g.R;  // the group is one contiguous range of the block
    wave_units(xp_from_load_count(g, k, gh), lane,
               [&](uint32_t v) { return UnitOffs{v * 16, xp_from_load_lds(g, k, v)}; },
               [&](uint32_t o) -> u32x4 { return *(const gu4*)(in + o); }, to_lds);
    wave_sync();
    if (k == 0)
      wave_units(xp_from_store_count(g, gh), lane,
                 [&](uint32_t u) { return UnitOffs{xp_from_store_lds(g, 0, gh, u), xp_from_store_dst(g, h0, gh, u)}; },
                 [&](uint32_t o) -> u32x4 { return *reinterpret_cast<const lu4*>(lds + o); }, to_dst);
    else
      wave_units(xp_from_store_count(g, gh), lane,
                 [&](uint32_t u) { return UnitOffs{xp_from_store_lds(g, 1, gh, u), xp_from_store_dst(g, h0, gh, u)}; },
                 [&](uint32_t o) -> u32x4 { return gather16<E>(lds + o, rs); }, to_dst);
    wave_sync();
  }
}

template <uint32_t E>
__device__ __forceinline__ void xpacked_piece(const uint8_t* src, uint8_t* dst, bool to_block, uint32_t k,
                                              const XGeom& g, lds_u8* lds, uint32_t lane, uint32_t first,
                                              uint32_t end) {
  if (to_block)
    xpacked_to_block<E>(src, dst, k, g, lds, lane, first, end);
  else
    xpacked_from_block<E>(src, dst, k, g, lds, lane, first, end);
}

// ---------------------------------------------------------------- head-major KV layout
// A paged-KV piece in the head-major (HND) layout: the block is [H][B][R], the
// host piece [B][H][R]. Whole rows move, so there is no LDS stage: units are
// taken in host order, which keeps the PCIe side (host reads of a fetch, host
// writes of an offload) contiguous, and the HBM side is read or written in whole
// rows (256 bytes for the 64k-token workload).
__device__ __forceinline__ void hnd_piece(const uint8_t* src, uint8_t* dst, bool to_block, const XGeom& g,
                                          uint32_t lane) {
  auto get = [&](uint32_t o) -> u32x4 { return *(const gu4*)(src + o); };
  auto put = [&](uint32_t o, u32x4 v) { *(gu4*)(dst + o) = v; };
  if (to_block)
    wave_units(hnd_count(g), lane, [&](uint32_t u) { return UnitOffs{u * 16, hnd_block_off(g, u)}; }, get, put);
  else
    wave_units(hnd_count(g), lane, [&](uint32_t u) { return UnitOffs{hnd_block_off(g, u), u * 16}; }, get, put);
}

// Template value of transfer_body for the head-major layout (the x-packed ones
// are the element sizes 1, 2, 4, 8).
constexpr uint32_t kXeHnd = 0x100;

extern __shared__ __attribute__((aligned(16))) uint8_t mma_dyn_lds[];

// The dummy-task kernel's body. kXE = 0: paged-KV blocks hold pieces as the
// host does. kXE = kXeHnd: head-major blocks (a row permutation, no LDS).
// kXE = element bytes: the x-packed GPU block layout through LDS --
// one kernel per element size, so that no launch carries the registers or LDS
// of a transform it does not run.
template <uint32_t kXE>
__device__ __forceinline__ void transfer_body(const KernelArgs& a) {
  __shared__ uint64_t s_layer[kMaxLayers];
  Record* rec = a.rec;
  DevState* ds = a.ds;
  const uint32_t lane = threadIdx.x & (kWave - 1);

  // KV layer table from the kernel arguments into LDS.
  const uint32_t nl = a.kv_layers < kMaxLayers ? a.kv_layers : kMaxLayers;
  for (uint32_t i = threadIdx.x; i < nl; i += kBlock) s_layer[i] = a.layer_ptr[i];
  const uint64_t piece = a.kv_piece_bytes;
  const uint64_t kstride = a.kv_kstride;
  const XGeom xg{a.kv_tokens, a.kv_heads, a.kv_row_bytes, a.kv_elem, a.kv_lds_wave};
  lds_u8* wave_lds = (lds_u8*)(mma_dyn_lds) + (threadIdx.x / kWave) * a.kv_lds_wave;
  __syncthreads();

  // One ring entry: words a, b and count | kind_p0 (see CuEntry). One copy site
  // for every kind (a linear entry is a single "piece"), so the copy loop is
  // instantiated once.
  auto run_entry = [&](uint64_t w1, uint64_t w2, uint64_t w3) {
    const uint32_t count = static_cast<uint32_t>(w3);
    const uint32_t kind = static_cast<uint32_t>(w3 >> 32) & kEntryKindMask;
    const uint32_t p0 = static_cast<uint32_t>(w3 >> 40);
    // Data landed by an SDMA engine during this kernel: drop any stale copy of
    // it from this CU's vector L1 (and non-coherent L2 lines) before reading.
    if ((w3 >> 32) & kEntryAcquire) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "");
    const bool paged = kind != kEntryCopy;
    const uint32_t npieces = paged ? count : 1u;
    for (uint32_t j = 0; j < npieces; ++j) {
      const uint8_t* src = reinterpret_cast<const uint8_t*>(w1);
      uint8_t* dst = reinterpret_cast<uint8_t*>(w2);
      uint64_t n = count;
      if (paged) {
        const uint32_t p = p0 + j;
        uint8_t* pg = reinterpret_cast<uint8_t*>(s_layer[p >> 1]) + (p & 1u) * kstride + w2 * piece;
        uint8_t* contig = reinterpret_cast<uint8_t*>(w1) + j * piece;
        src = kind == kEntryToPaged ? contig : pg;
        dst = kind == kEntryToPaged ? pg : contig;
        n = piece;
        if constexpr (kXE == kXeHnd) {
          hnd_piece(src, dst, kind == kEntryToPaged, xg, lane);
          continue;
        } else if constexpr (kXE != 0) {
          xpacked_piece<kXE>(src, dst, kind == kEntryToPaged, p & 1u, xg, wave_lds, lane, 0, xg.H);
          continue;
        }
      }
      wave_copy(src, dst, n, lane);
    }
  };

  // A self-contained launch of a whole KV transfer (linear ones use
  // mma_whole_kernel): wave w copies entry w of the arguments and writes its
  // done tag -- no start signal, record, ring or wait.
  if (a.self_contained) {
    const uint32_t w = blockIdx.x * kWavesPerWG + threadIdx.x / kWave;
    if (w < a.n_pre) {
      run_entry(a.pre[w][0], a.pre[w][1], a.pre[w][2]);
      if (a.release_each) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");
      if (lane == 0) st_sys(&a.done[w], make_tag(a.seq, w));
    }
    return;
  }

  // 1. start signal (stream -> engine). Work that precedes this kernel in
  // stream order is complete and visible (dispatch acquire/release).
  if (lane == 0) {
    const uint32_t first = __hip_atomic_fetch_add(&ds->arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (first == 0) st_sys(&rec->h.started, a.seq);
  }

  // 2. CU-path worker loop. Lane 0 claims; lanes 0..4 fetch the entry with one
  // load instruction; the wave copies.
  uint64_t hb = 0, t_prog = 0;
  uint32_t timed_out = 0;
  if (lane == 0) t_prog = wall_clock64();
  for (;;) {
    uint64_t x = 0;
    if (lane == 0)
      x = __hip_atomic_fetch_add(&ds->cursor, static_cast<uint64_t>(1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    x = lane_u64(x, 0);
    if (a.device_ctl && x >= a.n_total) break;  // the whole CU share was in the ring at launch
    const uint64_t expect = make_tag(a.seq, x);
    const uint64_t* ew = reinterpret_cast<const uint64_t*>(&rec->ring[x % kRingSize]);
    uint32_t state = 0;  // 1: entry ready, 3: watchdog
    uint64_t w1 = 0, w2 = 0, w3 = 0;
    if (x < a.n_pre) {  // first entries arrive with the launch: no PCIe round trip
      w1 = a.pre[x][0];
      w2 = a.pre[x][1];
      w3 = a.pre[x][2];
      state = 1;
    }
    for (uint32_t polls = 0; state == 0; ++polls) {
      const uint64_t w = lane < 5 ? ld_sys(ew + lane) : 0;
      if (lane_u64(w, 0) == expect && lane_u64(w, 4) == expect) {
        w1 = lane_u64(w, 1);
        w2 = lane_u64(w, 2);
        w3 = lane_u64(w, 3);
        state = 1;
        break;
      }
      if ((polls & 7) == 7) {  // watchdog check every 8th poll
        uint32_t st = 0;
        if (lane == 0) {
          const uint64_t now = wall_clock64();
          const uint64_t hb2 = ld_sys(&rec->h.heartbeat);
          if (hb2 != hb) {
            hb = hb2;
            t_prog = now;
          } else if (now - t_prog > a.watchdog_ticks ||
                     __hip_atomic_load(&ds->timed_out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
            st = 3;
          }
        }
        st = __builtin_amdgcn_readfirstlane(st);
        if (st) {
          state = st;
          break;
        }
      }
      backoff(polls < 4 ? 1u : (polls < 16 ? 4u : 8u));
    }
    if (state != 1) {
      if (state == 3) timed_out = 1;
      break;
    }
    if ((static_cast<uint32_t>(w3 >> 32) & kEntryKindMask) == kEntryEnd)
      break;  // the ring is closed and this ticket is past its end
    run_entry(w1, w2, w3);
    if (a.release_each) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");
    if (lane == 0) {
      st_sys(&a.done[x % kRingSize], expect);
      t_prog = wall_clock64();
    }
  }

  // 3. leave; the last wave out waits for completion of all paths.
  if (lane == 0) {
    if (timed_out) {
      __hip_atomic_store(&ds->timed_out, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const uint32_t n = __hip_atomic_fetch_add(&ds->exited, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    if (n == a.total_waves - 1) {
      uint32_t to = __hip_atomic_load(&ds->timed_out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      int32_t status = 0;
      if (a.device_ctl) {
        // Every wave has left, so the CU share has landed; the copy engines'
        // share has when their completion signal reaches 0. Nothing re-arms
        // the watchdog here: it runs from this wave's last completion.
        int64_t left = 0;
        while (!to && a.sdma_left &&
               (left = __hip_atomic_load(const_cast<int64_t*>(a.sdma_left), __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_SYSTEM)) > 0) {
          if (wall_clock64() - t_prog > a.watchdog_ticks) to = 1;
          __builtin_amdgcn_s_sleep(8);
        }
        if (left < 0) status = 2;
      } else {
        while (!to && ld_sys(&rec->h.complete) != a.seq) {
          const uint64_t now = wall_clock64();
          const uint64_t hb2 = ld_sys(&rec->h.heartbeat);
          if (hb2 != hb) {
            hb = hb2;
            t_prog = now;
          } else if (now - t_prog > a.watchdog_ticks) {
            to = 1;
          }
          __builtin_amdgcn_s_sleep(8);
        }
      }
      if (to) status = 1;
      if (status) __hip_atomic_store(&rec->h.status, status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      __hip_atomic_store(&ds->cursor, static_cast<uint64_t>(0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&ds->arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&ds->exited, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&ds->timed_out, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");
      st_sys(&rec->h.released, a.seq);
    }
  }
}

}  // namespace

__global__ __launch_bounds__(kBlock) void mma_transfer_kernel(KernelArgs a) { transfer_body<0>(a); }

// A self-contained launch: every entry of a linear transfer travels in the
// arguments and no copy engine takes part, so wave w of the grid copies entry w
// and writes its done tag -- no start signal, ring, exit count or wait. The
// arguments hold only the entries (N of them), so a deep queue of small
// transfers on one stream uses little of the runtime's kernel-argument pool.
template <uint32_t N>
__global__ __launch_bounds__(kBlock) void mma_whole_kernel(WholeArgs<N> a) {
  const uint32_t lane = threadIdx.x & (kWave - 1);
  const uint32_t w = blockIdx.x * kWavesPerWG + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  if (w >= a.n) return;
  wave_copy<true>(reinterpret_cast<const uint8_t*>(a.e[w][0]), reinterpret_cast<uint8_t*>(a.e[w][1]),
                  static_cast<uint32_t>(a.e[w][2]), lane);
  if (a.release_each) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");
  if (lane == 0) st_sys(&a.done[w], make_tag(a.seq, w));
}

__global__ __launch_bounds__(kBlock) void mma_transfer_hnd_kernel(KernelArgs a) { transfer_body<kXeHnd>(a); }

// ---------------------------------------------------------------- pool launches
// A paged-KV transfer between a pool and the paged layer tensors in one launch.
// With the pool in this GPU's memory it is bound by HBM: every byte is read once and written once, in the order
// of the destinations (mma_pool.h), with no ring and no host round trip.

// Source and destination address of a piece. word(i): word i of the arguments;
// kTab: the block table is in device memory instead.
struct PoolEnds {
  uint64_t from, to;
};
template <bool kTab, class Word>
__device__ __forceinline__ PoolEnds pool_ends(const PoolArgs& a, PoolPiece pp, Word word) {
  typedef __attribute__((address_space(1))) uint64_t gu64;
  uint64_t e;
  if constexpr (kTab)
    e = ((const gu64*)(a.tab))[pp.entry];
  else
    e = word(a.layers + pp.entry);
  const uint64_t pooled = a.pool + (e & 0xffffffffull) * a.slot_bytes + static_cast<uint64_t>(pp.p) * a.piece;
  const uint64_t paged = word(pp.p >> 1) + (pp.p & 1u) * a.kstride + (e >> 32) * a.piece;
  return PoolEnds{a.to_paged ? pooled : paged, a.to_paged ? paged : pooled};
}
__device__ __forceinline__ PoolEnds pool_ends(const PoolArgs& a, PoolPiece pp) {
  const auto word = [&](uint32_t i) { return a.w[i]; };
  return a.tab ? pool_ends<true>(a, pp, word) : pool_ends<false>(a, pp, word);
}
// Piece number q of the layers' keys (kind 0) or values (1).
__device__ __forceinline__ PoolPiece kind_piece(const PoolGeom& g, uint32_t q, uint32_t kind) {
  const PoolPiece pp = pool_piece(g, q);
  return PoolPiece{pp.entry, 2 * pp.p + kind};
}

// s_waitcnt vmcnt(0), the other counters left alone (gfx9 encoding).
constexpr int kWaitVm0 = 0x0f70;

// The counters of a pool launch (pool_last). landed() is a wait for the wave's own
// stores, which at this scope go to memory themselves: a release, which writes back
// the L2, cost a launch of one block 6 us.
struct DevCounters {
  uint32_t* c;
  __device__ __forceinline__ uint32_t add(uint32_t i) const {
    return __hip_atomic_fetch_add(c + i * kPoolCtrStride, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ void zero(uint32_t i) const {
    __hip_atomic_store(c + i * kPoolCtrStride, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ void landed() const {
    __builtin_amdgcn_s_waitcnt(kWaitVm0);
    __builtin_amdgcn_sched_barrier(0);
  }
};

// The start tag, where the other direction's engine thread looks for it.
__device__ __forceinline__ void pool_begin(const PoolArgs& a) {
  if (a.started && blockIdx.x == 0 && threadIdx.x == 0) st_sys(a.started, make_tag(a.seq, 0));
}

// The workgroup that finishes last writes the done tag. The counters only order
// the tag after every workgroup: the data itself becomes visible to later work
// through the stream, when the kernel ends, as for any kernel (a device-wide
// release per workgroup would write back the L2 of its XCD each time). Counts on
// one address go one after the other, some 12 ns each, so 32 workgroups and more
// count in groups of at least 16 first (pool_last): with 512 and more to a group a
// launch of 2048 took 8 us longer. A launch of many has its tag written by a launch of
// its own instead (kPoolTagLaunch).
__device__ __forceinline__ void pool_finish(const PoolArgs& a) {
  if (a.clear && blockIdx.x == 0 && threadIdx.x == 0)
    __hip_atomic_store(a.clear, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (!a.done) return;
  if (a.release) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");
  __syncthreads();
  if (threadIdx.x != 0) return;
  if (a.tags) {  // few workgroups: tags of their own, no count (an atomic's round trip, about 1 us)
    for (uint32_t t = blockIdx.x; t < a.tags; t += gridDim.x) st_sys(&a.done[t], make_tag(a.seq, t));
    return;
  }
  if (!pool_last(blockIdx.x, gridDim.x, a.claim != nullptr, kPoolCtrs, DevCounters{a.ctr})) return;
  if (a.release) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
  st_sys(a.done, make_tag(a.seq, 0));
}

__device__ __forceinline__ SpanWalk span_walk(const PoolArgs& a, uint32_t wave) {
  return span_walk(blockIdx.x, gridDim.x, wave, kWavesPerWG, a.link != 0);
}
// Before the span's own reads, so that the claim's round trip overlaps theirs.
__device__ __forceinline__ void span_claim(const PoolArgs& a, SpanWalk& s, uint32_t lane) {
  if (a.claim && lane == 0)
    s.got = __hip_atomic_fetch_add(a.claim, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void span_next(const PoolArgs& a, SpanWalk& s) {
  span_next(s, a.claim != nullptr, a.claim ? __builtin_amdgcn_readfirstlane(s.got) : 0);
}

// Aligned pieces in the piece layout or (kHnd) head-major: one 16-byte unit per
// lane. What hides the latency is the 32 waves a CU holds (the kernel takes few
// registers), not loads in flight per wave, and small waves keep the writes in
// order: 8 GiB fetch and offload 2.90 and 2.86 ms, 5.9 and 6.0 TB/s; with 32 KiB
// read per wave before it writes 2.96 and 2.87, and 5.5 against 6.1 TB/s at 1 GiB.
// Nontemporal: every byte is moved once, caching it would only evict other data.
// But reads (kNt) not where head rows end inside a 128-byte line, whose other part
// a neighbour reads: 160-byte rows, 1 GiB fetched in 431 us, nontemporally 492;
// 256-byte rows 393 and 375.
template <bool kHnd, bool kNt>
__global__ __launch_bounds__(kBlock) void mma_kv_pool_kernel(PoolArgs a) {
  const uint32_t lane = threadIdx.x & (kWave - 1);
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  for (uint64_t w = static_cast<uint64_t>(blockIdx.x) * kWavesPerWG + wave; w < a.g.waves;
       w += static_cast<uint64_t>(gridDim.x) * kWavesPerWG) {
    const PoolUnit x = pool_unit(a.g, static_cast<uint32_t>(w), lane);
    if (x.ok) {
      const PoolEnds e = pool_ends(a, pool_piece(a.g, x.q));
      const gu4* src = (const gu4*)(e.from) + (kHnd ? hnd_other(a.hnd, x.u) : x.u);
      __builtin_nontemporal_store(kNt ? __builtin_nontemporal_load(src) : *src, (gu4*)(e.to) + x.u);
    }
  }
  pool_finish(a);
}

// Pieces span by span (a.g counts a span as a row), in HBM or over the link:
// x-packed ones (kXE: element bytes) through the wave's LDS tile, whole or by heads,
// a.group at a time; kXE = 0, pieces or addresses that are no multiple of 16, by wave_copy.
template <uint32_t kXE>
__global__ __launch_bounds__(kBlock) void mma_kv_pool_span_kernel(PoolArgs a) {
  const uint32_t lane = threadIdx.x & (kWave - 1);
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const XGeom g{a.tokens, a.heads, a.row_bytes, a.elem, a.lds_wave};
  pool_begin(a);
  for (SpanWalk s = span_walk(a, wave); s.at * a.group < a.g.waves; span_next(a, s)) {
    span_claim(a, s, lane);
    const uint64_t end = min(a.g.waves, (s.at + 1) * a.group);
    for (uint64_t w = s.at * a.group; w < end; ++w) {
      const uint32_t q = div_by(a.g.rows, static_cast<uint32_t>(w));
      const PoolPiece pp = pool_piece(a.g, q);
      PoolEnds e = pool_ends(a, pp);
      e.from = lane_u64(e.from, 0);
      e.to = lane_u64(e.to, 0);
      const uint32_t part = static_cast<uint32_t>(w - static_cast<uint64_t>(q) * a.g.rows.d);
      if constexpr (kXE != 0) {
        const uint32_t h0 = part * a.span;
        xpacked_piece<kXE>(reinterpret_cast<const uint8_t*>(e.from), reinterpret_cast<uint8_t*>(e.to), a.to_paged,
                           pp.p & 1u, g, (lds_u8*)(mma_dyn_lds) + wave * a.lds_wave, lane, h0,
                           min(g.H, h0 + a.span));
      } else {
        const uint64_t off = static_cast<uint64_t>(part) * a.span;
        wave_copy(reinterpret_cast<const uint8_t*>(e.from + off), reinterpret_cast<uint8_t*>(e.to + off),
                  min(static_cast<uint64_t>(a.span), a.piece - off), lane);
      }
    }
  }
  pool_finish(a);
}

// x units of x elements each, transposed: unit j gets element j of every unit.
template <uint32_t E>
__device__ __forceinline__ void transpose_units(u32x4 (&v)[16 / E]) {
  constexpr uint32_t X = 16 / E;
  u32x4 o[X];
  if constexpr (E == 1) {
#pragma unroll
    for (uint32_t j = 0; j < X; ++j)
#pragma unroll
      for (uint32_t w = 0; w < 4; ++w) {
        const uint32_t s = (j & 3u) | ((j & 3u) + 4) << 8;  // byte j of either word
        const uint32_t lo = __builtin_amdgcn_perm(v[4 * w + 1][j / 4], v[4 * w][j / 4], s);
        const uint32_t hi = __builtin_amdgcn_perm(v[4 * w + 3][j / 4], v[4 * w + 2][j / 4], s);
        o[j][w] = __builtin_amdgcn_perm(hi, lo, 0x05040100u);
      }
  } else if constexpr (E == 2) {
#pragma unroll
    for (uint32_t j = 0; j < X; ++j)
#pragma unroll
      for (uint32_t w = 0; w < 4; ++w)
        o[j][w] = __builtin_amdgcn_perm(v[2 * w + 1][j / 2], v[2 * w][j / 2], j & 1u ? 0x07060302u : 0x05040100u);
  } else if constexpr (E == 4) {
#pragma unroll
    for (uint32_t j = 0; j < X; ++j)
#pragma unroll
      for (uint32_t w = 0; w < 4; ++w) o[j][w] = v[w][j];
  } else {
#pragma unroll
    for (uint32_t j = 0; j < X; ++j)
#pragma unroll
      for (uint32_t w = 0; w < 4; ++w) o[j][w] = v[w / 2][2 * j + w % 2];
  }
#pragma unroll
  for (uint32_t j = 0; j < X; ++j) v[j] = o[j];
}

// x-packed pieces, in HBM (kLink false: a row per wave) or over the link (as
// mma_kv_link_kernel): keys first, then values, both straight through registers
// (XpMap), so no LDS limits the waves in flight and small pieces share a wave.
// Where it is used and what it gains: xp_registers.
// kStage (in HBM, where xp_stages): the block side of the values goes through a
// tile of the wave in LDS, in whole rows of 1 KiB, where each lane by itself
// accesses 2 * B bytes of each of its x dimensions at a time. The tiles (8 KiB a
// wave for 2-byte elements, 16 for one byte) leave 20 and 8 waves a CU, so a wave
// reads 8 rows of keys at once, as over the link. Before (the faster of whole
// pieces through LDS and plain registers) / staged, fetch and offload, us:
//   2 GiB of 32 KiB pieces          828 / 813    872 / 845
//   1 GiB                           408 / 412    430 / 421
//   128 MiB                          54 / 45      56 / 47
//   1 GiB, one-byte elements        469 / 421    534 / 426
//   469 MiB, 32 tokens x 5 x 80     208 / 192    266 / 229
// (by call, on one box; 2 GiB fetched took 820 to 826 on others, the kernel alone 800).
// 1, 2 and 4 rows of keys: 2 GiB 1110, 879, 817 and 1092, 871, 846; one-byte
// elements -, 572, 459.
template <uint32_t E, bool kLink, bool kStage>
__global__ __launch_bounds__(kBlock) void mma_kv_pool_xp_kernel(PoolArgs a) {
  constexpr uint32_t X = 16 / E, K = xp_key_rows(kLink, kStage);
  __shared__ u32x4 s_tile[kStage ? kWavesPerWG * kWave * X : 1];
  const uint32_t lane = threadIdx.x & (kWave - 1);
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint64_t keys = span_count(a.g.waves, K);
  if constexpr (kLink) pool_begin(a);
  for (SpanWalk s = span_walk(a, wave); s.at < keys + a.gv.waves; span_next(a, s)) {
    span_claim(a, s, lane);
    if (s.at < keys) {
      const gu4* from[K];
      gu4* to[K];
#pragma unroll
      for (uint32_t k = 0; k < K; ++k) {
        const uint64_t row = s.at * K + k;
        const bool in = row < a.g.waves;
        const PoolUnit x = pool_unit(a.g, static_cast<uint32_t>(in ? row : s.at * K), lane);
        const bool ok = x.ok && in;
        const PoolEnds e = pool_ends(a, kind_piece(a.g, ok ? x.q : 0, 0));
        const XpAt p = xp_key(a.xp, ok ? x.u : 0);
        const uint32_t host = xp_host(a.xp, p.hc, p.t), blk = xp_key_block(a.xp, p.hc, p.t);
        from[k] = (const gu4*)(e.from + (a.to_paged ? host : blk));
        to[k] = ok ? (gu4*)(e.to + (a.to_paged ? blk : host)) : nullptr;
      }
      u32x4 v[K];
#pragma unroll
      for (uint32_t k = 0; k < K; ++k) v[k] = *from[k];
      __builtin_amdgcn_s_waitcnt(kWaitVm0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (uint32_t k = 0; k < K; ++k)
        if (to[k]) *to[k] = v[k];
    } else if constexpr (kStage) {
      const PoolUnit x = pool_unit(a.gv, static_cast<uint32_t>(s.at - keys), lane);
      const uint32_t first = __builtin_amdgcn_readfirstlane(x.u), n = min(kWave, a.gv.units - first) * X;
      const PoolEnds e = pool_ends(a, kind_piece(a.gv, __builtin_amdgcn_readfirstlane(x.q), 1));
      const XpAt p = xp_val(a.xp, x.ok ? x.u : first);
      const uint32_t host = xp_host(a.xp, p.hc, p.t * X), hstep = a.xp.HC * 16;
      const uint64_t blk = static_cast<uint64_t>(first) * X * 16;
      lu4* tile = (lu4*)(s_tile) + wave * kWave * X;
      u32x4 v[X];
      if (a.to_paged) {
        if (x.ok) {
#pragma unroll
          for (uint32_t i = 0; i < X; ++i)
            v[i] = *(const gu4*)(e.from + host + static_cast<uint64_t>(i) * hstep);
          transpose_units<E>(v);
#pragma unroll
          for (uint32_t i = 0; i < X; ++i) tile[xp_stage_at<X>(a.xp, xp_stage_unit<X>(a.xp, lane, i))] = v[i];
        }
        wave_sync();
#pragma unroll
        for (uint32_t k = 0; k < X; ++k) {
          const uint32_t u = k * kWave + lane;
          if (u < n) __builtin_nontemporal_store(tile[xp_stage_at<X>(a.xp, u)], (gu4*)(e.to + blk) + u);
        }
      } else {
#pragma unroll
        for (uint32_t k = 0; k < X; ++k) {
          const uint32_t u = k * kWave + lane;
          v[k] = __builtin_nontemporal_load((const gu4*)(e.from + blk) + (u < n ? u : 0));
        }
#pragma unroll
        for (uint32_t k = 0; k < X; ++k) tile[xp_stage_at<X>(a.xp, k * kWave + lane)] = v[k];
        wave_sync();
        if (x.ok) {
#pragma unroll
          for (uint32_t i = 0; i < X; ++i) v[i] = tile[xp_stage_at<X>(a.xp, xp_stage_unit<X>(a.xp, lane, i))];
          transpose_units<E>(v);
#pragma unroll
          for (uint32_t i = 0; i < X; ++i) *(gu4*)(e.to + host + static_cast<uint64_t>(i) * hstep) = v[i];
        }
      }
      wave_sync();  // before the next row overwrites the tile
    } else {
      const PoolUnit x = pool_unit(a.gv, static_cast<uint32_t>(s.at - keys), lane);
      if (x.ok) {
        const PoolEnds e = pool_ends(a, kind_piece(a.gv, x.q, 1));
        const XpAt p = xp_val(a.xp, x.u);
        // Element i of the host side's units is token p.t * X + i, of the block's
        // dimension p.hc * X + i.
        const uint32_t host = xp_host(a.xp, p.hc, p.t * X), hstep = a.xp.HC * 16;
        const uint32_t blk = xp_val_block(a.xp, p.hc * X, p.t), bstep = a.xp.groups.d * 16;
        const uint64_t src = e.from + (a.to_paged ? host : blk), dst = e.to + (a.to_paged ? blk : host);
        const uint32_t sstep = a.to_paged ? hstep : bstep, dstep = a.to_paged ? bstep : hstep;
        u32x4 v[X];
#pragma unroll
        for (uint32_t i = 0; i < X; ++i) v[i] = *(const gu4*)(src + static_cast<uint64_t>(i) * sstep);
        transpose_units<E>(v);
#pragma unroll
        for (uint32_t i = 0; i < X; ++i) *(gu4*)(dst + static_cast<uint64_t>(i) * dstep) = v[i];
      }
    }
  }
  pool_finish(a);
}

// The same pieces with the pool in pinned host memory: bound by the PCIe link, so
// few waves (the launch keeps to a limit of workgroups) with much in flight each.
// A wave takes span after span of kLinkRows rows (SpanWalk): all addresses first (from the words in
// LDS: the arguments are host memory), then all reads, then all writes. Rows count across pieces, so small
// pieces fill a wave as large ones do. Reads past the last row repeat a unit of
// piece 0. Over 64 MiB (36 layers of 2 KiB pieces / 32 layers of 32 KiB pieces):
// fetch 1192 / 1190 us, 56.3 GB/s, where the link needs 1171; through the ring,
// whose micro-tasks are no larger than a block, 4762 / 1211. Spans of 4 and 16 rows
// took 1195 and 1245 us, all with 24 workgroups.
// kShared: pieces below a row share one (each lane its own piece); else a row's
// piece is the same for all lanes and its addresses are scalars.
template <bool kHnd, bool kTab, bool kShared, class Word>
__device__ __forceinline__ void link_span(const PoolArgs& a, uint32_t first, uint32_t lane, Word word) {
  constexpr uint32_t K = kLinkRows;
  const gu4* from[K];
  gu4* to[K];
#pragma unroll
  for (uint32_t k = 0; k < K; ++k) {
    const bool in = first + k < a.g.waves;
    const PoolUnit x = pool_unit(a.g, in ? first + k : first, lane);
    const bool ok = x.ok && in;
    PoolEnds e;
    if constexpr (kShared) {
      e = pool_ends<kTab>(a, pool_piece(a.g, ok ? x.q : 0), word);
    } else {
      e = pool_ends<kTab>(a, pool_piece(a.g, __builtin_amdgcn_readfirstlane(x.q)), word);
      e.from = lane_u64(e.from, 0);
      e.to = lane_u64(e.to, 0);
    }
    const uint32_t u = ok ? x.u : 0, v = kHnd ? hnd_other(a.hnd, u) : u;
    from[k] = (const gu4*)(e.from) + (a.to_paged ? u : v);
    to[k] = ok ? (gu4*)(e.to) + (a.to_paged ? v : u) : nullptr;
  }
  u32x4 v[K];
#pragma unroll
  for (uint32_t k = 0; k < K; ++k) v[k] = *from[k];
  // All reads are in before the first write: left to itself the compiler, which
  // loses count of them over the branches below, waits before every write, and
  // so for the write before it too.
  __builtin_amdgcn_s_waitcnt(kWaitVm0);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (uint32_t k = 0; k < K; ++k)
    if (to[k]) *to[k] = v[k];
}

template <bool kHnd, bool kTab>
__global__ __launch_bounds__(kBlock) void mma_kv_link_kernel(PoolArgs a) {
  const uint32_t lane = threadIdx.x & (kWave - 1);
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  __shared__ uint64_t s_w[kPoolWords];
  pool_begin(a);
  for (uint32_t i = threadIdx.x; i < a.words; i += kBlock) s_w[i] = a.w[i];
  __syncthreads();
  const auto word = [&](uint32_t i) { return s_w[i]; };
  for (SpanWalk s = span_walk(a, wave); s.at * kLinkRows < a.g.waves; span_next(a, s)) {
    const uint64_t first = s.at * kLinkRows;
    span_claim(a, s, lane);
    if (a.g.per_row > 1)
      link_span<kHnd, kTab, true>(a, static_cast<uint32_t>(first), lane, word);
    else
      link_span<kHnd, kTab, false>(a, static_cast<uint32_t>(first), lane, word);
  }
  pool_finish(a);
}

// The done tag of a pool launch that does not count its workgroups: this launch
// starts when that one has ended.
__global__ void mma_kv_pool_tag_kernel(uint64_t* done, uint64_t tag) { st_sys(done, tag); }

// A pool launch's block table from the arena in host memory to its copy in
// device memory: 512 bytes per wave and read.
__global__ __launch_bounds__(kBlock) void mma_kv_pool_table_kernel(PoolTabArgs a) {
  const uint64_t i = static_cast<uint64_t>(blockIdx.x) * kBlock + threadIdx.x;
  if (i < a.n) a.to[i] = ld_sys(a.from + i);
}

template <uint32_t E>
__global__ __launch_bounds__(kBlock) void mma_transfer_xpacked_kernel(KernelArgs a) {
  transfer_body<E>(a);
}

// ------------------------------------------------------- KV fetch that allocates nothing
// Table chunk of a no-alloc KV fetch: entries [first, first + count) of the
// call's block table from the arguments into the scratch array.
__global__ __launch_bounds__(kBlock) void mma_kv_noalloc_table_kernel(NoallocTabArgs a) {
  uint64_t* tab = a.scratch + kNoallocTabOffset / 8;
  for (uint32_t j = threadIdx.x; j < a.count; j += kBlock) tab[a.first + j] = a.e[j];
}

// Claim words [0, n) of the scratch array to 0.
__global__ void mma_kv_noalloc_clear_kernel(uint32_t* w, uint32_t n) {
  for (uint32_t i = threadIdx.x; i < n; i += kWave)
    __hip_atomic_store(w + i, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// digest += sum_i (w_i + 1) * (2i + 1) mod 2^64 over nw words (+ one zero-padded
// tail word of tail_len bytes at tail). vec4: w is 16-byte aligned.
__global__ __launch_bounds__(256) void mma_digest_kernel(const uint32_t* __restrict__ w, uint64_t nw,
                                                         const uint8_t* __restrict__ tail, uint32_t tail_len,
                                                         uint32_t vec4, unsigned long long* out) {
  const uint64_t tid = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const uint64_t stride = static_cast<uint64_t>(gridDim.x) * blockDim.x;
  uint64_t acc = 0;
  uint64_t done = 0;
  if (vec4) {
    const uint64_t n4 = nw >> 2;
    const uint4* w4 = reinterpret_cast<const uint4*>(w);
    for (uint64_t j = tid; j < n4; j += stride) {
      const uint4 v = w4[j];
      const uint64_t i = j << 2;
      acc += (v.x + 1ull) * (2 * i + 1) + (v.y + 1ull) * (2 * i + 3) + (v.z + 1ull) * (2 * i + 5) +
             (v.w + 1ull) * (2 * i + 7);
    }
    done = n4 << 2;
  }
  for (uint64_t i = done + tid; i < nw; i += stride) acc += (w[i] + 1ull) * (2 * i + 1);
  if (tid == 0 && tail_len) {
    uint32_t t = 0;
    for (uint32_t b = 0; b < tail_len; ++b) t |= static_cast<uint32_t>(tail[b]) << (8 * b);
    acc += (t + 1ull) * (2 * nw + 1);
  }
  for (int off = kWave / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if ((threadIdx.x & (kWave - 1)) == 0 && acc) atomicAdd(out, static_cast<unsigned long long>(acc));
}

template <uint32_t N>
hipError_t launch_whole(const KernelArgs& args, uint32_t grid, hipStream_t stream) {
  WholeArgs<N> w;
  w.done = args.done;
  w.seq = args.seq;
  w.n = args.n_pre;
  w.release_each = args.release_each;
  for (uint32_t i = 0; i < args.n_pre; ++i)
    for (int k = 0; k < 3; ++k) w.e[i][k] = args.pre[i][k];
  void* params[] = {&w};
  return hipLaunchKernel(reinterpret_cast<const void*>(&mma_whole_kernel<N>), dim3(grid), dim3(kBlock), params, 0,
                         stream);
}

// Whether x-packed pieces that are not staged (xp_stages) go through registers
// (mma_kv_pool_xp_kernel) or through a wave's LDS tile, by what was faster (LDS /
// registers, us):
//  - pieces below 4 KiB, of which registers take several at a time: 64 MiB of 2 KiB
//    pieces over the link 1415 / 1221;
//  - in HBM small pieces of elements of two bytes and more: 1 GiB fetched of 4, 5 and 6
//    KiB pieces 658 / 490, 566 / 488, 503 / 486, 64 MiB 44 / 28, 38 / 28, 34 / 28;
//  - offloads in HBM, whose stores are whole rows of tokens: 1 GiB of 6 KiB pieces
//    531 / 504, of one-byte elements 985 / 652; only 24 tokens x 5 x 80 (557 / 620) and
//    48 x 8 x 128 (474 / 504) are the other way round, above 256 MiB;
//  - other fetches in HBM that are small. One-byte elements, 8 KiB pieces: 8 MiB 10.2 /
//    11.0, 64 MiB 30 / 40, 1 GiB 459 / 664. Token groups that are no power of two: 24
//    tokens x 8 x 128, 64 MiB 33 / 28, 126 MiB 63 / 59, 1 GiB 440 / 460; 48 x 8 x 128,
//    64 MiB 46 / 27, 252 MiB 139 / 119, 1 GiB 451 / 450; with more than 16 KiB of tile a
//    wave (one workgroup per CU), 48 x 8 x 256, 63 MiB 68 / 27, 252 MiB 159 / 116, 1 GiB
//    450 / 442;
//  - over the link fetches whose tile is above 16 KiB a wave: 1 block of 32 tokens
//    x 8 heads x 256 dimensions 306 / 267, but of 16 x 8 x 128 43.8 / 48.7; and
//    offloads below 16 MiB in 8 x 8 squares: 48.3 / 45.6, but with 50 units a token
//    175 / 186 at 8 MiB, and 64 MiB 1292 / 1361.
bool xp_registers(const PoolArgs& p, uint32_t n, bool link) {
  const uint64_t bytes = static_cast<uint64_t>(n) * 2 * p.layers * p.piece;
  if (p.piece < 4096 || (!link && p.elem > 1 && p.piece < 8192)) return true;
  if (!link) return !p.to_paged || bytes <= (p.lds_wave > 16 * 1024 ? 256ull << 20 : (p.elem > 1 ? 64ull : 8ull) << 20);
  if (p.to_paged) return p.lds_wave > 16 * 1024;
  return bytes < (16ull << 20) && p.tokens % 8 == 0 && p.heads * (p.row_bytes / 16) % 8 == 0;
}

// One launch of the kernel that the pool's place, the layout and the alignment
// ask for. p holds everything but the geometry; wgs: the most workgroups of a
// launch over the link, 0 for a pool in HBM.
hipError_t launch_pool_kernel(PoolArgs& p, uint32_t n, uint32_t layout, bool aligned, uint32_t wgs,
                              hipStream_t stream, bool* begun) {
  const uint32_t by_piece = wgs ? 0 : p.to_paged;
  uint32_t lds = 0;
  p.link = wgs ? 1 : 0;
  p.group = 1;
  p.g = pool_geom(n, 2 * p.layers, p.piece >> 4, by_piece);
  const void* k = nullptr;
  uint64_t spans = span_count(p.g.waves, wgs ? kLinkRows : 1);  // of one wave each
  const bool stage = !wgs && layout == kKvLayoutXPacked && xp_stages(p.piece, p.tokens, p.elem);
  if (layout == kKvLayoutHnd) {
    const bool heads_first = !wgs && p.to_paged;
    p.hnd = heads_first ? hnd_map(p.heads, p.tokens, p.row_bytes / 16) : hnd_map(p.tokens, p.heads, p.row_bytes / 16);
    k = !wgs ? (p.row_bytes % 128 == 0 ? reinterpret_cast<const void*>(&mma_kv_pool_kernel<true, true>)
                                       : reinterpret_cast<const void*>(&mma_kv_pool_kernel<true, false>))
        : p.tab ? reinterpret_cast<const void*>(&mma_kv_link_kernel<true, true>)
                : reinterpret_cast<const void*>(&mma_kv_link_kernel<true, false>);
  } else if (layout == kKvLayoutXPacked && !stage && !xp_registers(p, n, wgs != 0)) {
    lds = kWavesPerWG * p.lds_wave;
    k = p.elem == 1   ? reinterpret_cast<const void*>(&mma_kv_pool_span_kernel<1>)
        : p.elem == 2 ? reinterpret_cast<const void*>(&mma_kv_pool_span_kernel<2>)
        : p.elem == 4 ? reinterpret_cast<const void*>(&mma_kv_pool_span_kernel<4>)
                      : reinterpret_cast<const void*>(&mma_kv_pool_span_kernel<8>);
    // Claimed fetches go by the heads that fill the tile: with whole pieces the last
    // ones of few kept single waves busy. 192 pieces of 32 and 64 KiB 126 / 121 and
    // 250 / 236 us, 6 blocks of 4 MiB 488 / 457 (the entries of whole transfers: 121,
    // 239, 461). With fixed shares whole pieces are better: 3 MiB 66.8 / 71.3.
    p.span = p.claim && p.to_paged ? xp_to_heads(XGeom{p.tokens, p.heads, p.row_bytes, p.elem, p.lds_wave}) : p.heads;
    p.g.rows = fast_div((p.heads + p.span - 1) / p.span);
    p.g.waves = static_cast<uint64_t>(p.g.total) * p.g.rows.d;
    // A claim's round trip pays for 8 KiB at least; with few waves for more, as they
    // lose less at the end.
    const uint64_t bytes = p.piece / p.heads * p.span;
    if (p.claim)
      p.group = static_cast<uint32_t>(std::max<uint64_t>(1, (link_few(wgs) ? kLinkFewSpan : kPoolSpan) / bytes));
    spans = span_count(p.g.waves, p.group);
  } else if (layout == kKvLayoutXPacked) {
    const uint32_t x = 16 / p.elem, hc = p.heads * (p.row_bytes / 16);
    p.xp = xp_map(p.tokens, hc, x);
    p.g = pool_geom(n, p.layers, static_cast<uint64_t>(hc) * p.tokens, by_piece);
    p.gv = pool_geom(n, p.layers, static_cast<uint64_t>(hc) * (p.tokens / x), by_piece);
    spans = span_count(p.g.waves, xp_key_rows(wgs != 0, stage)) + p.gv.waves;
    const void* const xp[4][3] = {{reinterpret_cast<const void*>(&mma_kv_pool_xp_kernel<1, false, false>),
                                   reinterpret_cast<const void*>(&mma_kv_pool_xp_kernel<1, true, false>),
                                   reinterpret_cast<const void*>(&mma_kv_pool_xp_kernel<1, false, true>)},
                                  {reinterpret_cast<const void*>(&mma_kv_pool_xp_kernel<2, false, false>),
                                   reinterpret_cast<const void*>(&mma_kv_pool_xp_kernel<2, true, false>),
                                   reinterpret_cast<const void*>(&mma_kv_pool_xp_kernel<2, false, true>)},
                                  {reinterpret_cast<const void*>(&mma_kv_pool_xp_kernel<4, false, false>),
                                   reinterpret_cast<const void*>(&mma_kv_pool_xp_kernel<4, true, false>),
                                   reinterpret_cast<const void*>(&mma_kv_pool_xp_kernel<4, false, true>)},
                                  {reinterpret_cast<const void*>(&mma_kv_pool_xp_kernel<8, false, false>),
                                   reinterpret_cast<const void*>(&mma_kv_pool_xp_kernel<8, true, false>),
                                   reinterpret_cast<const void*>(&mma_kv_pool_xp_kernel<8, false, true>)}};
    k = xp[p.elem == 1 ? 0 : p.elem == 2 ? 1 : p.elem == 4 ? 2 : 3][wgs ? 1 : stage ? 2 : 0];
  } else if (aligned && !link_long_spans(wgs, p.piece)) {
    k = !wgs ? reinterpret_cast<const void*>(&mma_kv_pool_kernel<false, true>)
        : p.tab ? reinterpret_cast<const void*>(&mma_kv_link_kernel<false, true>)
                : reinterpret_cast<const void*>(&mma_kv_link_kernel<false, false>);
  } else {
    p.span = link_few(wgs) ? kLinkFewSpan : wgs ? 2 * kPoolSpan : kPoolSpan;
    const uint64_t per = (p.piece + p.span - 1) / p.span;
    p.g.rows = fast_div(static_cast<uint32_t>(per));
    spans = p.g.waves = per * p.g.total;
    k = reinterpret_cast<const void*>(&mma_kv_pool_span_kernel<0>);
  }
  const uint64_t grid = pool_grid(spans, kWavesPerWG, wgs);
  uint64_t* const done = p.done;
  if (grid > kPoolTagLaunch) p.done = nullptr;
  void* params[] = {&p};
  const hipError_t e = hipLaunchKernel(k, dim3(static_cast<uint32_t>(grid)), dim3(kBlock), params, lds, stream);
  if (e != hipSuccess) return e;
  *begun = true;
  if (p.done == done) return e;
  uint64_t* d = done;
  uint64_t tag = make_tag(p.seq, 0);
  void* tag_params[] = {&d, &tag};
  return hipLaunchKernel(reinterpret_cast<const void*>(&mma_kv_pool_tag_kernel), dim3(1), dim3(1), tag_params, 0,
                         stream);
}

hipError_t launch_pool(const KernelArgs& args, hipStream_t stream, bool* begun) {
  static thread_local PoolArgs p;
  p.done = args.done;
  p.seq = args.seq;
  p.ctr = args.pool_ctr;
  p.tab = nullptr;
  p.pool = args.pool_base;
  p.piece = args.kv_piece_bytes;
  p.slot_bytes = p.piece * 2 * args.kv_layers;
  p.kstride = args.kv_kstride;
  p.to_paged = args.pool_to_paged;
  p.layers = args.kv_layers;
  p.tokens = args.kv_tokens;
  p.heads = args.kv_heads;
  p.row_bytes = args.kv_row_bytes;
  p.elem = args.kv_elem;
  // Stores to a host pool are in host memory before the done tag; in HBM the
  // stream orders them (a release per wave writes back its XCD's L2 each time).
  p.release = args.pool_link && args.release_each;
  p.lds_wave = args.kv_lds_wave;
  uint64_t mis = p.piece | p.pool;
  for (uint32_t l = 0; l < p.layers; ++l) mis |= p.w[l] = args.layer_ptr[l];
  p.words = p.layers;
  p.tags = args.pool_link && !args.pool_claim ? args.pool_wgs : 0;
  p.claim = args.pool_claim ? args.pool_ctr + kPoolCtrStride : nullptr;
  p.clear = nullptr;
  p.started = args.pool_started;
  if (p.layers + args.pool_blocks <= kPoolWords) {
    p.words += static_cast<uint32_t>(args.pool_blocks);
    memcpy(p.w + p.layers, args.pool_tab_host, args.pool_blocks * sizeof(uint64_t));
  } else {
    PoolTabArgs t{args.pool_tab, args.pool_tab_copy, args.pool_blocks};
    void* params[] = {&t};
    const hipError_t e =
        hipLaunchKernel(reinterpret_cast<const void*>(&mma_kv_pool_table_kernel),
                        dim3(static_cast<uint32_t>((t.n + kBlock - 1) / kBlock)), dim3(kBlock), params, 0, stream);
    if (e != hipSuccess) return e;
    *begun = true;
    p.tab = args.pool_tab_copy;
  }
  return launch_pool_kernel(p, static_cast<uint32_t>(args.pool_blocks), args.kv_layout, (mis & 15u) == 0,
                            args.pool_link ? args.pool_wgs : 0, stream, begun);
}

// begun: set once a launch of the transfer is on the stream, also when a later
// one of the same transfer fails.
hipError_t launch_transfer(const KernelArgs& args, uint32_t grid, hipStream_t stream, bool* begun) {
  if (args.pool_tab) return launch_pool(args, stream, begun);
  if (args.self_contained && args.kv_layers == 0) {  // linear: the lean kernel; KV: below, by layout
    if (args.n_pre <= 4) return launch_whole<4>(args, grid, stream);
    if (args.n_pre <= 16) return launch_whole<16>(args, grid, stream);
    return launch_whole<kPrefill>(args, grid, stream);
  }
  void* params[] = {const_cast<KernelArgs*>(&args)};
  // Only x-packed KV transfers stage through LDS; every other launch asks for
  // none, so it can share CUs with kernels that use most of theirs.
  if (args.kv_layout == kKvLayoutXPacked) {
    const void* k = args.kv_elem == 1   ? reinterpret_cast<const void*>(&mma_transfer_xpacked_kernel<1>)
                    : args.kv_elem == 2 ? reinterpret_cast<const void*>(&mma_transfer_xpacked_kernel<2>)
                    : args.kv_elem == 4 ? reinterpret_cast<const void*>(&mma_transfer_xpacked_kernel<4>)
                                        : reinterpret_cast<const void*>(&mma_transfer_xpacked_kernel<8>);
    return hipLaunchKernel(k, dim3(grid), dim3(kBlock), params, kWavesPerWG * args.kv_lds_wave, stream);
  }
  if (args.kv_layout == kKvLayoutHnd)
    return hipLaunchKernel(reinterpret_cast<const void*>(&mma_transfer_hnd_kernel), dim3(grid), dim3(kBlock), params,
                           0, stream);
  return hipLaunchKernel(reinterpret_cast<const void*>(&mma_transfer_kernel), dim3(grid), dim3(kBlock), params, 0,
                         stream);
}

hipError_t launch_digest(const void* ptr, uint64_t bytes, uint64_t* out, hipStream_t stream) {
  const uint32_t* w = static_cast<const uint32_t*>(ptr);
  uint64_t nw = bytes >> 2;
  const uint8_t* tail = static_cast<const uint8_t*>(ptr) + (nw << 2);
  uint32_t tail_len = static_cast<uint32_t>(bytes & 3u);
  uint32_t vec4 = (reinterpret_cast<uintptr_t>(ptr) & 15u) == 0 ? 1u : 0u;
  unsigned long long* o = reinterpret_cast<unsigned long long*>(out);
  uint64_t want = (nw + 4095) / 4096;
  uint32_t grid = static_cast<uint32_t>(want < 1 ? 1 : (want > 2048 ? 2048 : want));
  void* params[] = {&w, &nw, &tail, &tail_len, &vec4, &o};
  return hipLaunchKernel(reinterpret_cast<const void*>(&mma_digest_kernel), dim3(grid), dim3(256), params, 0,
                         stream);
}


// ------------------------------------------------------- KV fetch that allocates nothing
// The no-alloc KV fetch's claim words and block table: a fixed array of this
// library's device code, so that the call needs no allocation. Every GPU the
// library runs on holds its own copy, at its own address, until the process
// ends. In host code the array's name is only a stand-in: its device address
// is looked up once per device (noalloc_setup, called by mma_init with that
// device current) and only that address is used.
static __device__ __align__(256) uint8_t scratch[kNoallocScratchBytes];

namespace {
uint64_t* g_scratch_dev[kNoallocDevices] = {};
}  // namespace

hipError_t noalloc_setup(int dev) {
  if (dev < 0 || dev >= kNoallocDevices) return hipErrorInvalidDevice;
  if (g_scratch_dev[dev]) return hipSuccess;
  void* p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return e;
  if (!p || (reinterpret_cast<uintptr_t>(p) & 255u) != 0) return hipErrorInvalidSymbol;
  g_scratch_dev[dev] = static_cast<uint64_t*>(p);
  return hipSuccess;
}

uint64_t* noalloc_scratch(int dev) { return dev >= 0 && dev < kNoallocDevices ? g_scratch_dev[dev] : nullptr; }

hipError_t launch_noalloc_table(const NoallocTabArgs& t, hipStream_t stream) {
  void* params[] = {const_cast<NoallocTabArgs*>(&t)};
  return hipLaunchKernel(reinterpret_cast<const void*>(&mma_kv_noalloc_table_kernel), dim3(1), dim3(kBlock), params,
                         0, stream);
}

hipError_t launch_noalloc_clear(uint32_t* w, uint32_t n, hipStream_t stream) {
  void* params[] = {&w, &n};
  return hipLaunchKernel(reinterpret_cast<const void*>(&mma_kv_noalloc_clear_kernel), dim3(1), dim3(kWave), params, 0,
                         stream);
}

hipError_t launch_noalloc(PoolArgs& p, uint32_t n, uint32_t layout, uint32_t wgs, hipStream_t stream) {
  uint64_t mis = p.piece | p.pool;
  for (uint32_t l = 0; l < p.layers; ++l) mis |= p.w[l];
  bool begun = false;  // this call's scratch is never given back
  return launch_pool_kernel(p, n, layout, (mis & 15u) == 0, wgs, stream, &begun);
}

}  // namespace mma
