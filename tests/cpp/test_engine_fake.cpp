// CPU test of the host engine on fake paths (no GPU). The engine code under
// test is the product's (mma_engine.h): planner output, path selector,
// copy-engine slots with merging, CU-ring protocol, completion and retirement.
// Only the GPU side is replaced:
//   - FakeBackend: "copy engines" are host threads that run commands in order,
//     each taking bytes / rate plus a fixed per-command cost, then memcpy and
//     drop the command's signal to 0;
//   - the dummy-task kernel is emulated by host threads ("waves") that follow
//     the record protocol of mma_proto.h: claim tickets with an atomic cursor,
//     wait for tagged ring entries, copy (at a per-wave rate), write done tags,
//     and the last wave out waits for `complete`, resets the device state and
//     releases the record;
//   - "device memory" is host memory.
// Scenarios: byte-exact results for copies, tensor lists and paged-KV fetch /
// offload through staging; every micro-task retired exactly once; a slower
// copy engine receives proportionally fewer micro-tasks; merged commands;
// submit failures re-routed; two streams in flight; and pull-based selection
// against the best fixed split at 1:1 and 2:1 path-rate ratios (the paper's
// static-split comparison, Section 5.1.2). Built twice by the pytest wrapper:
// optimised, and with ThreadSanitizer (correctness scenarios only).
//
// Usage: test_engine_fake [--no-timing | --timing-only]
// The timing scenarios sleep to emulate path rates, so a heavily loaded host
// distorts them; the pytest wrapper runs them apart from the correctness ones.
#include <array>
#include <atomic>
#include <chrono>
#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <future>
#include <mutex>
#include <random>
#include <thread>
#include <vector>

#include "mma_engine.h"

using namespace mma;

namespace {

int g_failures = 0;
#define CHECK(cond, ...)                                          \
  do {                                                            \
    if (!(cond)) {                                                \
      ++g_failures;                                               \
      std::printf("FAIL %s:%d: %s -- ", __FILE__, __LINE__, #cond); \
      std::printf(__VA_ARGS__);                                   \
      std::printf("\n");                                          \
    }                                                             \
  } while (0)

void sleep_ns(uint64_t ns) {
  if (ns) std::this_thread::sleep_for(std::chrono::nanoseconds(ns));
}

// ------------------------------------------------------------ fake backend
class FakeBackend final : public Backend {
 public:
  // rate in bytes per microsecond (1000 = 1 GB/s), cost per command in ns
  FakeBackend(std::vector<double> rates, uint64_t cmd_ns) : cmd_ns_(cmd_ns) {
    for (double r : rates) {
      auto e = std::make_unique<Eng>();
      e->rate = r;
      engines_.push_back(std::move(e));
    }
    for (auto& e : engines_) {
      Eng* p = e.get();
      p->th = std::thread([this, p] { run(p); });
    }
  }
  ~FakeBackend() override {
    for (auto& e : engines_) {
      {
        std::lock_guard<std::mutex> g(e->mu);
        e->stop = true;
      }
      e->cv.notify_all();
      e->th.join();
    }
  }
  mma_status_t alloc_records(uint64_t bytes, void** host, void** dev) override {
    *host = *dev = std::aligned_alloc(4096, (bytes + 4095) & ~4095ull);
    return *host ? MMA_OK : MMA_ERR_NO_MEMORY;
  }
  void free_records(void* host) override {
    frees_.fetch_add(1);
    std::free(host);
  }
  int frees() const { return frees_.load(); }
  mma_status_t alloc_device_state(uint64_t bytes, void** dev) override {
    *dev = std::aligned_alloc(128, (bytes + 127) & ~127ull);
    if (!*dev) return MMA_ERR_NO_MEMORY;
    std::memset(*dev, 0, bytes);
    return MMA_OK;
  }
  void free_device_state(void* dev) override {
    frees_.fetch_add(1);
    std::free(dev);
  }
  mma_status_t alloc_host_scratch(uint64_t bytes, void** host) override {
    *host = std::calloc(1, bytes);
    return *host ? MMA_OK : MMA_ERR_NO_MEMORY;
  }
  void free_host_scratch(void* host) override { std::free(host); }
  bool signal_create(uint64_t* sig) override {
    *sig = reinterpret_cast<uint64_t>(new std::atomic<int64_t>(1));
    return true;
  }
  void signal_destroy(uint64_t sig) override { delete reinterpret_cast<std::atomic<int64_t>*>(sig); }
  void signal_store(uint64_t sig, int64_t v) override {
    reinterpret_cast<std::atomic<int64_t>*>(sig)->store(v, std::memory_order_release);
  }
  int64_t signal_load(uint64_t sig) override {
    return reinterpret_cast<std::atomic<int64_t>*>(sig)->load(std::memory_order_acquire);
  }
  bool signal_create_polled(uint64_t* sig, const int64_t** value) override {
    if (!polled_) return false;
    auto* a = new std::atomic<int64_t>(0);
    *sig = reinterpret_cast<uint64_t>(a);
    *value = reinterpret_cast<const int64_t*>(a);
    return true;
  }
  void signal_sub(uint64_t sig, int64_t v) override {
    reinterpret_cast<std::atomic<int64_t>*>(sig)->fetch_sub(v, std::memory_order_acq_rel);
  }
  void set_polled(bool on) { polled_ = on; }
  bool copy(int engine, void* dst, bool, const void* src, bool, uint64_t bytes, uint64_t sig) override {
    if (engine < 0 || engine >= static_cast<int>(engines_.size())) return false;
    Eng* e = engines_[engine].get();
    {
      std::lock_guard<std::mutex> g(e->mu);
      e->q.push_back({dst, src, bytes, sig, 0});
      e->pending.fetch_add(1);
      e->bytes_total += bytes;
      e->commands += 1;
    }
    e->cv.notify_all();
    return true;
  }
  // Another component's command on engine e (not this library's): it keeps the
  // engine busy for hold_ns and signals nothing.
  void foreign(int e, uint64_t hold_ns) {
    Eng* p = engines_[e].get();
    {
      std::lock_guard<std::mutex> g(p->mu);
      p->q.push_back({nullptr, nullptr, 0, 0, hold_ns});
      p->pending.fetch_add(1);
    }
    p->cv.notify_all();
  }
  uint32_t engines_idle(int) override {
    uint32_t m = 0;
    for (size_t i = 0; i < engines_.size(); ++i)
      if (engines_[i]->pending.load() == 0) m |= 1u << i;
    return m;
  }
  uint64_t engine_bytes(int e) {
    std::lock_guard<std::mutex> g(engines_[e]->mu);
    return engines_[e]->bytes_total;
  }

 private:
  struct Cmd {
    void* dst;
    const void* src;
    uint64_t bytes;
    uint64_t sig;
    uint64_t hold_ns;  // foreign work: no copy, no signal
  };
  struct Eng {
    double rate = 1000;
    std::mutex mu;
    std::condition_variable cv;
    std::deque<Cmd> q;
    std::atomic<int> pending{0};
    uint64_t bytes_total = 0, commands = 0;
    bool stop = false;
    std::thread th;
  };
  void run(Eng* e) {
    for (;;) {
      Cmd c;
      {
        std::unique_lock<std::mutex> lk(e->mu);
        e->cv.wait(lk, [&] { return e->stop || !e->q.empty(); });
        if (e->q.empty()) return;
        c = e->q.front();
        e->q.pop_front();
      }
      if (c.hold_ns) {
        sleep_ns(c.hold_ns);
        e->pending.fetch_sub(1);
        continue;
      }
      // the command lands after its modelled time; the host's memcpy runs inside it
      const auto end = std::chrono::steady_clock::now() +
                       std::chrono::nanoseconds(cmd_ns_ + static_cast<uint64_t>(c.bytes * 1000.0 / e->rate));
      std::memcpy(c.dst, c.src, c.bytes);
      std::this_thread::sleep_until(end);
      e->pending.fetch_sub(1);
      signal_sub(c.sig, 1);  // a landed command decrements its signal
    }
  }
  uint64_t cmd_ns_;
  bool polled_ = true;
  std::atomic<int> frees_{0};
  std::vector<std::unique_ptr<Eng>> engines_;
};

// ------------------------------------------------------------ fake GPU stream
// Kernels on one stream run one after another; each is a set of wave threads.
class FakeStream {
 public:
  FakeStream() : th_([this] { run(); }) {}
  ~FakeStream() {
    {
      std::lock_guard<std::mutex> g(mu_);
      stop_ = true;
    }
    cv_.notify_all();
    th_.join();
  }
  void launch(std::function<void()> k) {
    {
      std::lock_guard<std::mutex> g(mu_);
      q_.push_back(std::move(k));
      ++pending_;
    }
    cv_.notify_all();
  }
  void synchronize() {
    std::unique_lock<std::mutex> lk(mu_);
    done_cv_.wait(lk, [&] { return pending_ == 0; });
  }

 private:
  void run() {
    for (;;) {
      std::function<void()> k;
      {
        std::unique_lock<std::mutex> lk(mu_);
        cv_.wait(lk, [&] { return stop_ || !q_.empty(); });
        if (q_.empty()) return;
        k = std::move(q_.front());
        q_.pop_front();
      }
      k();
      {
        std::lock_guard<std::mutex> g(mu_);
        --pending_;
      }
      done_cv_.notify_all();
    }
  }
  std::mutex mu_;
  std::condition_variable cv_, done_cv_;
  std::deque<std::function<void()>> q_;
  int pending_ = 0;
  bool stop_ = false;
  std::thread th_;
};

// One wave of the dummy-task kernel, following the record protocol.
template <class T>
T aload(const T* p) {
  return __atomic_load_n(p, __ATOMIC_ACQUIRE);
}
template <class T>
void astore(T* p, T v) {
  __atomic_store_n(p, v, __ATOMIC_RELEASE);
}

void copy_at_rate(void* dst, const void* src, uint64_t n, double wave_rate) {
  sleep_ns(static_cast<uint64_t>(n * 1000.0 / wave_rate));
  std::memcpy(dst, src, n);
}

// A pool launch of aligned pieces in the piece layout, as the runtime makes it of its
// arguments: the table in them or in its copy in device memory, the split of mma_pool.h,
// and a done tag per workgroup, or one by the workgroup that counts itself last or by a
// launch after it.
struct FakePool {
  KernelArgs a;
  std::vector<uint64_t> tab;  // as the arguments carry it
  bool copied;                // it does not fit them
  PoolGeom g;
  uint32_t grid;
};
struct FakeCounters {
  uint32_t* c;
  uint32_t add(uint32_t i) const { return __atomic_fetch_add(c + i * kPoolCtrStride, 1u, __ATOMIC_ACQ_REL); }
  void zero(uint32_t i) const { __atomic_store_n(c + i * kPoolCtrStride, 0u, __ATOMIC_RELEASE); }
  void landed() const {}
};
void pool_row(const FakePool& p, uint32_t w) {
  const KernelArgs& a = p.a;
  const uint64_t piece = a.kv_piece_bytes, slot_bytes = 2ull * a.kv_layers * piece;
  for (uint32_t lane = 0; lane < kWave; ++lane) {
    const PoolUnit u = pool_unit(p.g, w, lane);
    if (!u.ok) continue;
    const PoolPiece pp = pool_piece(p.g, u.q);
    const uint64_t e = p.copied ? a.pool_tab_copy[pp.entry] : p.tab[pp.entry];
    uint8_t* pooled = reinterpret_cast<uint8_t*>(a.pool_base + (e & 0xffffffffull) * slot_bytes + pp.p * piece + u.u * 16ull);
    uint8_t* paged = reinterpret_cast<uint8_t*>(a.layer_ptr[pp.p >> 1] + (pp.p & 1u) * a.kv_kstride + (e >> 32) * piece + u.u * 16ull);
    if (a.pool_to_paged)
      std::memcpy(paged, pooled, 16);
    else
      std::memcpy(pooled, paged, 16);
  }
}
void pool_workgroup(const FakePool& p, uint32_t wg) {
  const KernelArgs& a = p.a;
  const bool link = a.pool_link != 0, claims = a.pool_claim != 0;
  const uint32_t per = link ? kLinkRows : 1;
  FakeCounters ctr{a.pool_ctr};
  for (uint32_t wave = 0; wave < kWavesPerWG; ++wave) {
    SpanWalk s = span_walk(wg, p.grid, wave, kWavesPerWG, link);
    while (s.at < span_count(p.g.waves, per)) {
      const uint32_t got = claims ? ctr.add(1) : 0;
      for (uint64_t w = s.at * per; w < std::min<uint64_t>(p.g.waves, (s.at + 1) * per); ++w)
        pool_row(p, static_cast<uint32_t>(w));
      span_next(s, claims, got);
    }
  }
  if (link && !claims) {
    for (uint32_t t = wg; t < a.pool_wgs; t += p.grid) astore(&a.done[t], make_tag(a.seq, t));
    return;
  }
  if (p.grid <= kPoolTagLaunch && pool_last(wg, p.grid, claims, kPoolCtrs, ctr)) astore(&a.done[0], make_tag(a.seq, 0));
}

// Launches over the link that start wait here until it is false.
std::atomic<bool> g_hold_links{false};

// On the fake stream: a few host threads share its workgroups.
void pool_launch(FakeStream& st, const KernelArgs& a) {
  auto p = std::make_shared<FakePool>();
  p->a = a;
  const uint32_t n = static_cast<uint32_t>(a.pool_blocks);
  p->copied = a.kv_layers + a.pool_blocks > kPoolWords;
  if (!p->copied) p->tab.assign(a.pool_tab_host, a.pool_tab_host + n);
  p->g = pool_geom(n, 2 * a.kv_layers, a.kv_piece_bytes >> 4, a.pool_link ? 0 : a.pool_to_paged);
  p->grid = static_cast<uint32_t>(
      pool_grid(span_count(p->g.waves, a.pool_link ? kLinkRows : 1), kWavesPerWG, a.pool_link ? a.pool_wgs : 0));
  st.launch([p, n] {
    if (p->a.pool_started) astore(p->a.pool_started, make_tag(p->a.seq, 0));
    while (p->a.pool_link && g_hold_links) sleep_ns(100000);
    if (p->copied) std::memcpy(p->a.pool_tab_copy, p->a.pool_tab, n * sizeof(uint64_t));
    const uint32_t nt = std::min<uint32_t>(p->grid, 4);
    std::vector<std::thread> ts;
    for (uint32_t t = 0; t < nt; ++t)
      ts.emplace_back([&p, t, nt] {
        for (uint32_t wg = t; wg < p->grid; wg += nt) pool_workgroup(*p, wg);
      });
    for (auto& t : ts) t.join();
    if (p->grid > kPoolTagLaunch) astore(&p->a.done[0], make_tag(p->a.seq, 0));
  });
}

void wave(const KernelArgs a, uint32_t w, double wave_rate) {
  Record* rec = a.rec;
  DevState* ds = a.ds;
  const bool sc = a.self_contained != 0;
  if (!sc && __atomic_fetch_add(&ds->arrived, 1u, __ATOMIC_RELAXED) == 0) astore(&rec->h.started, a.seq);
  uint64_t hb = 0, t_prog = now_ns();
  bool timed_out = false, sc_taken = false;
  for (;;) {
    uint64_t x;
    if (sc) {
      if (sc_taken) break;
      sc_taken = true;
      x = w;
      if (x >= a.n_pre) break;
    } else {
      x = __atomic_fetch_add(&ds->cursor, 1ull, __ATOMIC_RELAXED);
      if (a.device_ctl && x >= a.n_total) break;
    }
    const uint64_t expect = make_tag(a.seq, x);
    uint64_t w1, w2, w3;
    if (x < a.n_pre) {
      w1 = a.pre[x][0];
      w2 = a.pre[x][1];
      w3 = a.pre[x][2];
    } else {
      CuEntry* e = &rec->ring[x % kRingSize];
      bool ready = false;
      while (!ready) {
        if (aload(&e->tag0) == expect && aload(&e->tag1) == expect) {
          ready = true;
          break;
        }
        const uint64_t hb2 = aload(&rec->h.heartbeat);
        if (hb2 != hb) {
          hb = hb2;
          t_prog = now_ns();
        } else if (now_ns() - t_prog > a.watchdog_ticks || __atomic_load_n(&ds->timed_out, __ATOMIC_RELAXED)) {
          break;
        }
        std::this_thread::yield();
      }
      if (!ready) {
        timed_out = true;
        break;
      }
      w1 = e->a;
      w2 = e->b;
      w3 = static_cast<uint64_t>(e->count) | (static_cast<uint64_t>(e->kind_p0) << 32);
    }
    const uint32_t count = static_cast<uint32_t>(w3);
    const uint32_t kind = static_cast<uint32_t>(w3 >> 32) & kEntryKindMask;
    if (kind == kEntryEnd) break;
    const uint32_t p0 = static_cast<uint32_t>(w3 >> 40);
    if (kind == kEntryCopy) {
      copy_at_rate(reinterpret_cast<void*>(w2), reinterpret_cast<const void*>(w1), count, wave_rate);
    } else {
      for (uint32_t j = 0; j < count; ++j) {
        const uint32_t p = p0 + j;
        uint8_t* pg = reinterpret_cast<uint8_t*>(a.layer_ptr[p >> 1]) + (p & 1u) * a.kv_kstride + w2 * a.kv_piece_bytes;
        uint8_t* contig = reinterpret_cast<uint8_t*>(w1) + j * a.kv_piece_bytes;
        if (kind == kEntryToPaged)
          copy_at_rate(pg, contig, a.kv_piece_bytes, wave_rate);
        else
          copy_at_rate(contig, pg, a.kv_piece_bytes, wave_rate);
      }
    }
    astore(&a.done[x % kRingSize], expect);
    t_prog = now_ns();
  }
  if (sc) return;
  if (timed_out) __atomic_store_n(&ds->timed_out, 1u, __ATOMIC_RELAXED);
  const uint32_t n = __atomic_fetch_add(&ds->exited, 1u, __ATOMIC_ACQ_REL);
  if (n == a.total_waves - 1) {
    bool to = __atomic_load_n(&ds->timed_out, __ATOMIC_RELAXED) != 0;
    int32_t status = 0;
    if (a.device_ctl) {
      int64_t left = 0;
      while (!to && a.sdma_left && (left = aload(a.sdma_left)) > 0) {
        if (now_ns() - t_prog > a.watchdog_ticks) to = true;
        std::this_thread::yield();
      }
      if (left < 0) status = 2;
    } else {
      while (!to && aload(&rec->h.complete) != a.seq) {
        const uint64_t hb2 = aload(&rec->h.heartbeat);
        if (hb2 != hb) {
          hb = hb2;
          t_prog = now_ns();
        } else if (now_ns() - t_prog > a.watchdog_ticks) {
          to = true;
        }
        std::this_thread::yield();
      }
    }
    if (to) status = 1;
    if (status) astore(&rec->h.status, status);
    __atomic_store_n(&ds->cursor, 0ull, __ATOMIC_RELAXED);
    __atomic_store_n(&ds->arrived, 0u, __ATOMIC_RELAXED);
    __atomic_store_n(&ds->exited, 0u, __ATOMIC_RELAXED);
    __atomic_store_n(&ds->timed_out, 0u, __ATOMIC_RELAXED);
    astore(&rec->h.released, a.seq);
  }
}

// ------------------------------------------------------------ harness
struct Setup {
  std::vector<double> engine_rates{2000, 2000};  // bytes/us
  double wave_rate = 250;                          // bytes/us per wave
  uint64_t cmd_ns = 20000;
  uint32_t mask = MMA_PATH_CU | 0x3;
  uint32_t mask_d2h = 0;  // device-to-host paths, when not `mask`
  uint32_t duplex[2] = {0, 0};  // paths while the other direction moves (0: the direction's own)
  Config cfg{};
};

Config default_config() {
  Config c{};
  c.chunk = 256 * 1024;
  c.fallback = 2 * c.chunk;
  c.small = 16 * 1024;
  c.sub = 64 * 1024;
  c.depth = 2;
  c.cu_depth = 4;
  c.backoff = 2;
  c.cu_wgs = 2;
  c.watchdog_ms = 20000;
  c.mask[0] = c.mask[1] = MMA_PATH_CU | 0x3;
  c.static_split = 0;
  c.static_cu_percent = 0;
  c.merge = 4;
  return c;
}

class Harness {
 public:
  explicit Harness(const Setup& s) : s_(s), be_(s.engine_rates, s.cmd_ns) {
    Config c = s.cfg;
    c.mask[MMA_H2D] = s.mask;
    c.mask[MMA_D2H] = s.mask_d2h ? s.mask_d2h : s.mask;
    for (int d = 0; d < 2; ++d) c.duplex[d] = s.duplex[d] ? s.duplex[d] : c.mask[d];
    stage_bytes_ = std::max<uint64_t>(c.chunk, 2 * 1024 * 1024);
    const uint32_t engines = 16;  // staging for any engine set
    staging_.assign(2 * engines * c.depth * stage_bytes_ + 1, 0);
    for (int d = 0; d < 2; ++d) {
      eng_[d].reset(new Engine(d, c, &be_, &stats_));
      void* base = staging_.data() + d * engines * c.depth * stage_bytes_;
      const mma_status_t rc = eng_[d]->init((c.mask[d] | c.duplex[d]) & 0xFFFFu, stage_bytes_, base);
      CHECK(rc == MMA_OK, "engine init %d: %s", rc, t_err.c_str());
    }
    eng_[MMA_D2H]->set_peer(eng_[MMA_H2D].get());  // as mma_init
    eng_[MMA_H2D]->set_peer(eng_[MMA_D2H].get());
    cfg_ = c;
  }
  ~Harness() {
    for (auto& e : eng_) e->shutdown();  // each engine thread reads the other's counters
    for (auto& e : eng_) e.reset();
  }
  // The runtime's submit(), with the fake stream in place of the kernel launch.
  // early: the stream is taken to be idle, so the transfer goes to the engine
  // before the launch (the copy engines may start at once); with launch =
  // false the launch then "fails" and the transfer is marked unlaunched.
  void submit(std::unique_ptr<Transfer> x, uint64_t payload, FakeStream& st, const KvGeom* kv = nullptr,
              bool early = false, bool launch = true) {
    Engine* e = eng_[x->dir].get();
    std::lock_guard<std::mutex> g(submit_mu_);
    CHECK(e->acquire(x.get(), payload, kv != nullptr, 60000), "record");
    KernelArgs a;
    const uint32_t grid = e->prepare(x.get(), ++seq_, payload, kv, 20000ull * 1000000ull, a);
    const uint32_t waves = grid * kWavesPerWG;
    const double rate = s_.wave_rate;
    Transfer* raw = x.get();
    if (early && !x->self_contained) {
      x->early = true;
      e->submit(std::move(x));
    }
    if (!launch) {
      if (x && x->light >= 0) {
        e->release_unused(x.get());
        return;
      }
      raw->unlaunched.store(true, std::memory_order_release);
      return;
    }
    if (a.pool_tab) {
      pool_launch(st, a);
    } else {
      st.launch([a, waves, rate] {
        std::vector<std::thread> ts;
        for (uint32_t w = 0; w < waves; ++w) ts.emplace_back(wave, a, w, rate);
        for (auto& t : ts) t.join();
      });
    }
    if (!x) return;
    if (x->light >= 0)
      e->track(std::move(x));  // as the runtime: whole transfers never reach the engine thread
    else
      e->submit(std::move(x));
  }
  // The runtime's submit() under device control: light (whole) transfers and
  // transfers that fit a ring are planned in full and launched; the engine
  // thread never sees them. Others fall back to submit(). idle: the stream is
  // taken to have nothing pending; launch = false: the launch "fails".
  void submit_device(std::unique_ptr<Transfer> x, uint64_t payload, FakeStream& st, const KvGeom* kv, bool idle,
                     bool launch = true) {
    Engine* e = eng_[x->dir].get();
    std::unique_lock<std::mutex> g(submit_mu_);
    CHECK(e->acquire(x.get(), payload, kv != nullptr, 60000), "record");
    KernelArgs a;
    const uint64_t wd = 20000ull * 1000000ull;
    const uint32_t grid = x->light >= 0 ? e->prepare(x.get(), ++seq_, payload, kv, wd, a)
                                        : e->prepare_device(x.get(), ++seq_, payload, kv, wd, idle, a);
    if (!grid) {  // too many micro-tasks for a ring: the engine thread takes it
      e->release_unused(x.get());
      x->rec = nullptr;
      x->light = -1;
      g.unlock();
      submit(std::move(x), payload, st, kv);
      return;
    }
    if (!launch) {
      if (x->light >= 0)
        e->release_unused(x.get());
      else
        e->abandon_device(x.get(), 60000);
      return;
    }
    const uint32_t waves = grid * kWavesPerWG;
    const double rate = s_.wave_rate;
    if (a.pool_tab) {
      pool_launch(st, a);
    } else {
      st.launch([a, waves, rate] {
        std::vector<std::thread> ts;
        for (uint32_t w = 0; w < waves; ++w) ts.emplace_back(wave, a, w, rate);
        for (auto& t : ts) t.join();
      });
    }
    e->track(std::move(x));
  }
  bool sync() { return eng_[0]->wait_idle(60000) && eng_[1]->wait_idle(60000); }
  const Config& cfg() const { return cfg_; }
  Stats& stats() { return stats_; }
  FakeBackend& backend() { return be_; }
  Engine* engine(int d) { return eng_[d].get(); }

 private:
  Setup s_;
  FakeBackend be_;
  Stats stats_;
  std::unique_ptr<Engine> eng_[2];
  std::vector<uint8_t> staging_;
  uint64_t stage_bytes_ = 0;
  Config cfg_{};
  std::mutex submit_mu_;
  uint64_t seq_ = 0;
};

std::vector<uint8_t> random_bytes(size_t n, uint32_t seed) {
  std::vector<uint8_t> v(n);
  std::mt19937 r(seed);
  for (auto& b : v) b = static_cast<uint8_t>(r());
  return v;
}

uint64_t sum_tasks(Stats& s, int from, int to) {
  uint64_t t = 0;
  for (int i = from; i < to; ++i) t += s.path_tasks[i].load();
  return t;
}

std::unique_ptr<Transfer> linear(int dir, void* dst, const void* src, uint64_t n, const Config& c) {
  mma_copy_desc_t d{dst, src, n};
  const uint64_t s = reinterpret_cast<uint64_t>(src), t = reinterpret_cast<uint64_t>(dst);
  return make_list_transfer(dir, &d, 1, &n, &s, &t, c);
}

// ------------------------------------------------------------ scenarios
// nap_ns > 0: the engine thread naps between rounds; the fake paths are slow,
// so the nap bounds assume a 1 GB/s link instead of 50.
void copies_are_exact(uint32_t mask, const char* name, bool early = false, uint64_t nap_ns = 0) {
  Setup s;
  s.cfg = default_config();
  s.cfg.nap_ns = nap_ns;
  s.cfg.overdue_gbs = nap_ns ? 1 : 0;
  s.mask = mask;
  Harness h(s);
  FakeStream st;
  for (int dir = 0; dir < 2; ++dir) {
    for (uint64_t n : {1ull, 777ull, 64ull * 1024, 300ull * 1024 + 5, 3ull * 1024 * 1024 + 123,
                       nap_ns ? 8ull * 1024 * 1024 + 9 : 0ull}) {
      if (!n) continue;
      auto src = random_bytes(n, static_cast<uint32_t>(n + dir));
      std::vector<uint8_t> dst(n + 64, 0xA5);
      auto x = linear(dir, dst.data() + 32, src.data(), n, h.cfg());
      const size_t tasks = x->tasks.size();
      const uint64_t before = sum_tasks(h.stats(), 0, MMA_NUM_PATHS);
      h.submit(std::move(x), n, st, nullptr, early);
      st.synchronize();
      CHECK(h.sync(), "sync");
      CHECK(std::memcmp(dst.data() + 32, src.data(), n) == 0, "%s dir=%d n=%llu: bytes differ", name, dir,
            (unsigned long long)n);
      CHECK(dst[31] == 0xA5 && dst[32 + n] == 0xA5, "%s: bytes outside the destination changed", name);
      CHECK(sum_tasks(h.stats(), 0, MMA_NUM_PATHS) - before == tasks, "%s: tasks retired %llu != %zu", name,
            (unsigned long long)(sum_tasks(h.stats(), 0, MMA_NUM_PATHS) - before), tasks);
    }
  }
  CHECK(h.stats().failed.load() == 0, "%s: failed transfers", name);
  CHECK(!nap_ns || h.stats().naps.load() > 0, "%s: the engine thread never napped", name);
  std::printf("ok   copies exact, every micro-task retired once (%s): cu tasks %llu, sdma tasks %llu, naps %llu\n",
              name, (unsigned long long)h.stats().path_tasks[16].load(), (unsigned long long)sum_tasks(h.stats(), 0, 16),
              (unsigned long long)h.stats().naps.load());
}

void list_with_merging() {
  Setup s;
  s.cfg = default_config();
  s.mask = 0x3;  // copy engines only: every micro-task goes through a command
  Harness h(s);
  FakeStream st;
  std::vector<uint64_t> sizes = {5, 300 * 1024, 1024 * 1024 + 17, 0, 70 * 1024, 2 * 1024 * 1024};
  uint64_t total = 0;
  for (auto z : sizes) total += z;
  auto src = random_bytes(total, 7);
  std::vector<uint8_t> dst(total, 0);
  std::vector<mma_copy_desc_t> list;
  std::vector<uint64_t> s_cu, d_cu;
  uint64_t off = 0;
  for (auto z : sizes) {  // back to back on both sides: runs cross tensor boundaries
    list.push_back({dst.data() + off, src.data() + off, z});
    s_cu.push_back(reinterpret_cast<uint64_t>(src.data() + off));
    d_cu.push_back(reinterpret_cast<uint64_t>(dst.data() + off));
    off += z;
  }
  auto x = make_list_transfer(MMA_H2D, list.data(), list.size(), sizes.data(), s_cu.data(), d_cu.data(), h.cfg());
  const size_t tasks = x->tasks.size();
  h.submit(std::move(x), total, st);
  st.synchronize();
  CHECK(h.sync(), "sync");
  CHECK(std::memcmp(dst.data(), src.data(), total) == 0, "list bytes differ");
  const uint64_t cmds = h.stats().sdma_commands.load();
  const uint64_t sdma_tasks = sum_tasks(h.stats(), 0, 16);
  CHECK(sdma_tasks + h.stats().path_tasks[16].load() == tasks, "tasks retired");
  CHECK(cmds < sdma_tasks, "merging: %llu commands for %llu micro-tasks", (unsigned long long)cmds,
        (unsigned long long)sdma_tasks);
  std::printf("ok   tensor list, merged commands: %llu commands for %llu copy-engine micro-tasks\n",
              (unsigned long long)cmds, (unsigned long long)sdma_tasks);
}

void kv_roundtrip(uint32_t mask, const char* name, bool early = false, uint64_t nap_ns = 0) {
  Setup s;
  s.cfg = default_config();
  s.cfg.chunk = 8 * 1024;  // 4 pieces per micro-task
  s.cfg.nap_ns = nap_ns;
  s.cfg.overdue_gbs = nap_ns ? 1 : 0;
  s.mask = mask;
  Harness h(s);
  FakeStream st;
  const uint32_t L = 3, ppb = 2 * L, slots = 24, nb = 30;
  const uint64_t piece = 2048, slot_bytes = piece * ppb;
  std::vector<uint8_t> pool = random_bytes(slots * slot_bytes, 11);
  std::vector<std::vector<uint8_t>> layers(L, std::vector<uint8_t>(2 * nb * piece, 0xA5));
  KvGeom kv;
  kv.piece = piece;
  kv.kstride = piece * nb;
  kv.layers = L;
  for (uint32_t l = 0; l < L; ++l) kv.layer_ptr[l] = reinterpret_cast<uint64_t>(layers[l].data());
  std::vector<int32_t> hs = {5, 0, 17, 3, 22, 9, 11, 1, 14, 20}, gb = {2, 29, 7, 0, 13, 21, 4, 26, 9, 15};
  const uint64_t host = reinterpret_cast<uint64_t>(pool.data());
  const bool sdma_ok = (mask & 0xFFFFu) != 0;
  auto x = make_kv_transfer(MMA_H2D, piece, ppb, host, host, false, sdma_ok, hs.data(), gb.data(), hs.size(), h.cfg());
  h.submit(std::move(x), hs.size() * slot_bytes, st, &kv, early);
  st.synchronize();
  CHECK(h.sync(), "sync");
  bool ok = true;
  for (size_t i = 0; i < hs.size(); ++i)
    for (uint32_t l = 0; l < L; ++l)
      for (uint32_t k = 0; k < 2; ++k)
        ok &= std::memcmp(layers[l].data() + (k * nb + gb[i]) * piece,
                          pool.data() + hs[i] * slot_bytes + (2 * l + k) * piece, piece) == 0;
  size_t untouched = 0;
  for (uint32_t l = 0; l < L; ++l)
    for (uint32_t k = 0; k < 2; ++k)
      for (uint32_t b = 0; b < nb; ++b)
        if (std::find(gb.begin(), gb.end(), static_cast<int32_t>(b)) == gb.end())
          untouched += layers[l][(k * nb + b) * piece] == 0xA5 && layers[l][(k * nb + b + 1) * piece - 1] == 0xA5;
  CHECK(ok, "%s: fetched pieces differ", name);
  CHECK(untouched == L * 2 * (nb - hs.size()), "%s: untouched blocks changed", name);
  // offload the same blocks into other slots
  std::vector<int32_t> dest = {23, 2, 4, 6, 8, 10, 12, 13, 15, 16};
  auto before = pool;
  auto y = make_kv_transfer(MMA_D2H, piece, ppb, host, host, false, sdma_ok, dest.data(), gb.data(), gb.size(),
                            h.cfg());
  h.submit(std::move(y), gb.size() * slot_bytes, st, &kv, early);
  st.synchronize();
  CHECK(h.sync(), "sync");
  auto want = before;
  for (size_t j = 0; j < gb.size(); ++j)
    for (uint32_t l = 0; l < L; ++l)
      for (uint32_t k = 0; k < 2; ++k)
        std::memcpy(want.data() + dest[j] * slot_bytes + (2 * l + k) * piece,
                    layers[l].data() + (k * nb + gb[j]) * piece, piece);
  CHECK(pool == want, "%s: offloaded pool differs", name);
  CHECK(h.stats().failed.load() == 0, "%s: failed", name);
  std::printf("ok   paged-KV fetch and offload (%s): staging bytes %llu, sdma commands %llu\n", name,
              (unsigned long long)h.stats().staging_bytes.load(), (unsigned long long)h.stats().sdma_commands.load());
}

// Transfers up to cfg.whole bytes whose micro-tasks fit one launch are taken
// whole by the CU path: self-contained launches, no copy-engine command, one
// wave per entry, at most kPrefill entries; larger ones still use every path.
void whole_transfers_on_cu() {
  Setup s;
  s.cfg = default_config();
  s.cfg.whole[0] = s.cfg.whole[1] = 4 * 1024 * 1024;
  s.mask = MMA_PATH_CU | 0x3;
  Harness h(s);
  FakeStream st;
  for (int dir = 0; dir < 2; ++dir) {
    for (uint64_t n : {1ull, 100000ull, 3ull * 1024 * 1024 + 7, 4ull * 1024 * 1024}) {
      auto src = random_bytes(n, static_cast<uint32_t>(n + 3 * dir));
      std::vector<uint8_t> dst(n + 64, 0xA5);
      const uint64_t cmds = h.stats().sdma_commands.load();
      auto x = linear(dir, dst.data() + 32, src.data(), n, h.cfg());
      h.submit(std::move(x), n, st);
      st.synchronize();
      CHECK(h.sync(), "sync");
      CHECK(std::memcmp(dst.data() + 32, src.data(), n) == 0, "whole dir=%d n=%llu: bytes differ", dir,
            (unsigned long long)n);
      CHECK(dst[31] == 0xA5 && dst[32 + n] == 0xA5, "whole: bytes outside the destination changed");
      CHECK(h.stats().sdma_commands.load() == cmds, "whole dir=%d n=%llu: a copy engine took part", dir,
            (unsigned long long)n);
    }
  }
  CHECK(h.stats().busy_ns.load() == 0, "whole transfers woke the engine thread");
  // Above the limit every path takes part again.
  const uint64_t n = 6 * 1024 * 1024;
  auto src = random_bytes(n, 99);
  std::vector<uint8_t> dst(n, 0);
  h.submit(linear(MMA_H2D, dst.data(), src.data(), n, h.cfg()), n, st);
  st.synchronize();
  CHECK(h.sync(), "sync");
  CHECK(dst == src, "6 MiB copy differs");
  CHECK(h.stats().sdma_commands.load() > 0, "above the whole-transfer limit the copy engines take part");
  CHECK(h.stats().failed.load() == 0, "whole: failed transfers");
  std::printf("ok   transfers up to the whole-transfer limit run as self-contained CU launches, retired without the "
              "engine thread\n");
}

// Small paged-KV fetches and offloads taken whole by the CU path: one
// self-contained launch each (entries in the arguments), exact, no copy-engine
// command, no engine-thread work; a larger one still uses every path.
void whole_kv_transfers() {
  Setup s;
  s.cfg = default_config();
  s.cfg.chunk = 8 * 1024;  // 4 pieces per micro-task
  s.cfg.whole[0] = s.cfg.whole[1] = 64 * 1024;
  Harness h(s);
  FakeStream st;
  const uint32_t L = 2, ppb = 2 * L, slots = 40, nb = 48;
  const uint64_t piece = 2048, slot_bytes = piece * ppb;  // 8 KiB slots
  std::vector<uint8_t> pool = random_bytes(slots * slot_bytes, 51);
  std::vector<std::vector<uint8_t>> layers(L, std::vector<uint8_t>(2 * nb * piece, 0xA5));
  KvGeom kv;
  kv.piece = piece;
  kv.kstride = piece * nb;
  kv.layers = L;
  for (uint32_t l = 0; l < L; ++l) kv.layer_ptr[l] = reinterpret_cast<uint64_t>(layers[l].data());
  const uint64_t host = reinterpret_cast<uint64_t>(pool.data());
  for (int n : {1, 3, 8, 20}) {  // 8, 24, 64 and 160 KiB: the last is above the whole-transfer limit
    std::vector<int32_t> hs(n), gb(n);
    for (int i = 0; i < n; ++i) {
      hs[i] = (7 * i + 3) % static_cast<int>(slots);
      gb[i] = (5 * i + 1) % static_cast<int>(nb);
    }
    const uint64_t cmds = h.stats().sdma_commands.load();
    h.submit(make_kv_transfer(MMA_H2D, piece, ppb, host, host, false, true, hs.data(), gb.data(), n, h.cfg()),
             n * slot_bytes, st, &kv);
    st.synchronize();
    CHECK(h.sync(), "sync");
    bool ok = true;
    for (int i = 0; i < n; ++i)
      for (uint32_t l = 0; l < L; ++l)
        for (uint32_t k = 0; k < 2; ++k)
          ok &= std::memcmp(layers[l].data() + (k * nb + gb[i]) * piece,
                            pool.data() + hs[i] * slot_bytes + (2 * l + k) * piece, piece) == 0;
    CHECK(ok, "whole KV fetch of %d blocks differs", n);
    const bool whole = n * slot_bytes <= 64 * 1024;
    if (whole) CHECK(h.stats().sdma_commands.load() == cmds, "whole KV fetch of %d blocks used a copy engine", n);
    if (!whole) CHECK(h.stats().sdma_commands.load() > cmds, "a KV fetch above the limit used no copy engine");
    // offload the same blocks into other slots
    std::vector<int32_t> dest(n);
    for (int i = 0; i < n; ++i) dest[i] = (hs[i] + 1) % static_cast<int>(slots);
    std::vector<bool> taken(slots, false);
    bool distinct = true;
    for (int i = 0; i < n; ++i) distinct &= !taken[dest[i]], taken[dest[i]] = true;
    if (!distinct) continue;
    auto want = pool;
    for (int j = 0; j < n; ++j)
      for (uint32_t l = 0; l < L; ++l)
        for (uint32_t k = 0; k < 2; ++k)
          std::memcpy(want.data() + dest[j] * slot_bytes + (2 * l + k) * piece,
                      layers[l].data() + (k * nb + gb[j]) * piece, piece);
    h.submit(make_kv_transfer(MMA_D2H, piece, ppb, host, host, false, true, dest.data(), gb.data(), n, h.cfg()),
             n * slot_bytes, st, &kv);
    st.synchronize();
    CHECK(h.sync(), "sync");
    CHECK(pool == want, "whole KV offload of %d blocks: pool differs", n);
  }
  CHECK(h.stats().failed.load() == 0, "whole KV: failed transfers");
  std::printf("ok   small KV fetches and offloads taken whole by the CU path; larger ones use every path\n");
}

// Which KV transfers with a pool on the host are one launch over the link, where both
// routes were measured (link_eligible).
struct LinkCase {
  int dir;
  uint32_t layout;
  uint64_t piece;
  uint32_t layers, blocks, wgs;
  bool link;
  uint64_t chunk = 2 * MiB;
};
void link_routes(const char* name, const std::vector<LinkCase>& cases) {
  for (const LinkCase& k : cases) {
    Setup s;
    s.cfg = default_config();
    s.cfg.chunk = k.chunk;
    s.cfg.whole[MMA_H2D] = 24 * MiB;
    s.cfg.whole[MMA_D2H] = 8 * MiB;
    s.cfg.cu_wgs = k.wgs;
    Harness h(s);
    KvGeom kv;
    kv.piece = k.piece;
    kv.layers = k.layers;
    kv.layout = k.layout;
    std::vector<int32_t> hs(k.blocks), gb(k.blocks);
    for (uint32_t i = 0; i < k.blocks; ++i) hs[i] = gb[i] = static_cast<int32_t>(i);
    const uint64_t slot = 2 * k.layers * k.piece;
    const std::unique_ptr<Transfer> x =
        make_kv_transfer(k.dir, k.piece, 2 * k.layers, 1 << 20, 1 << 20, false, true, hs.data(), gb.data(), k.blocks, h.cfg());
    CHECK(h.engine(k.dir)->link_eligible(x.get(), kv, k.blocks * slot, slot) == k.link,
          "%s: dir %d layout %u, %u blocks of %llu KiB in %llu KiB pieces, %u workgroups: expected %d", name, k.dir, k.layout,
          k.blocks, static_cast<unsigned long long>(slot / KiB), static_cast<unsigned long long>(k.piece / KiB), k.wgs, k.link);
  }
  std::printf("ok   route of KV transfers over the link: %s\n", name);
}
const uint32_t kP = kKvLayoutPiece, kX = kKvLayoutXPacked, kH = kKvLayoutHnd;
const std::vector<LinkCase> kFewWorkgroups = {
    {MMA_H2D, kX, 32 * KiB, 32, 10, 1, false}, {MMA_H2D, kX, 32 * KiB, 32, 10, 16, true},
    {MMA_H2D, kH, 8 * KiB, 24, 5, 2, false},   {MMA_H2D, kH, 8 * KiB, 24, 5, 16, true},
    {MMA_D2H, kP, 8 * KiB, 24, 18, 2, false},  {MMA_D2H, kP, 8 * KiB, 24, 18, 16, true},
    {MMA_H2D, kP, 2 * KiB, 12, 42, 1, false},  {MMA_H2D, kP, 2 * KiB, 12, 3, 1, true},
    {MMA_H2D, kH, 32 * KiB, 4, 2048, 3, false}, {MMA_H2D, kH, 32 * KiB, 4, 2048, 8, true},
    {MMA_H2D, kX, 4 * KiB, 24, 700, 2, false}, {MMA_H2D, kX, 4 * KiB, 24, 700, 4, true},
    {MMA_H2D, kP, 32 * KiB, 4, 2048, 1, true}, {MMA_H2D, kH, 2 * KiB, 16, 8192, 1, true},
    {MMA_H2D, kP, 2 * KiB, 16, 8192, 1, true}, {MMA_D2H, kH, 8 * KiB, 24, 53, 2, true},
};
const std::vector<LinkCase> kFewLarge = {
    {MMA_H2D, kP, 16 * KiB, 24, 7, 16, false}, {MMA_H2D, kP, 12800, 24, 4, 16, false}, {MMA_H2D, kP, 28 * KiB, 24, 2, 16, false},
    {MMA_H2D, kP, 8 * KiB, 24, 18, 16, true},  {MMA_H2D, kP, 16 * KiB, 24, 30, 16, true}, {MMA_H2D, kP, 10 * KiB, 24, 2, 16, true},
    {MMA_D2H, kP, 16 * KiB, 24, 7, 16, false}, {MMA_D2H, kP, 12 * KiB, 24, 7, 16, true},
    {MMA_H2D, kH, 16 * KiB, 24, 7, 16, true},  {MMA_H2D, kX, 32 * KiB, 32, 3, 16, true},
    {MMA_H2D, kP, 32 * KiB, 1, 40, 16, false}, {MMA_H2D, kP, 32 * KiB, 1, 100, 16, true},  // 100 blocks are too many entries
};
const std::vector<LinkCase> kChunks = {
    {MMA_H2D, kP, 32 * KiB, 32, 256, 16, false, 8 * MiB}, {MMA_H2D, kP, 32 * KiB, 16, 512, 16, true, 8 * MiB},
    {MMA_D2H, kP, 32 * KiB, 16, 512, 16, false, 8 * MiB}, {MMA_D2H, kP, 32 * KiB, 8, 1024, 16, true, 8 * MiB},
    {MMA_H2D, kP, 32 * KiB, 16, 512, 16, true, 512 * KiB}, {MMA_D2H, kX, 32 * KiB, 4, 2048, 16, true, 512 * KiB},
    {MMA_H2D, kP, 32 * KiB, 32, 256, 16, false},          {MMA_D2H, kP, 32 * KiB, 16, 512, 16, false},
};

// KV transfers between a pool in device memory and the paged layers (piece
// layout) run as pool launches: one launch, table from the arena, no ring and
// no copy engine. Pieces of 8 KiB + 48 bytes end in a short row. Launches
// queued back to back on one stream reuse light slots and counters. So does a launch
// over the link, with a done tag per workgroup and with claims. With the
// stream held, a transfer whose table finds no room in the arena takes the
// ring path instead, and all of them land once the stream runs.
void hbm_pool_launches() {
  Setup s;
  s.cfg = default_config();
  Harness h(s);
  for (const bool dev : {true, false}) {
    FakeStream st;
    const uint32_t L = 2, ppb = 2 * L, slots = 620, nb = 640;
    const uint64_t piece = 8192 + 48, slot_bytes = piece * ppb;
    std::vector<uint8_t> pool = random_bytes(slots * slot_bytes, 61);
    std::vector<std::vector<uint8_t>> layers(L, std::vector<uint8_t>(2 * nb * piece, 0xA5));
    KvGeom kv;
    kv.piece = piece;
    kv.kstride = piece * nb;
    kv.layers = L;
    for (uint32_t l = 0; l < L; ++l) kv.layer_ptr[l] = reinterpret_cast<uint64_t>(layers[l].data());
    const uint64_t base = reinterpret_cast<uint64_t>(pool.data());
    const uint64_t cmds = h.stats().sdma_commands.load();
    // 600 blocks do not fit the arguments, and their fetch over the link claims spans
    CHECK(link_claims(MMA_H2D, kKvLayoutPiece, 600 * slot_bytes) && 600 + L > kPoolWords, "sizes");
    const auto launch = [&](int dir, const std::vector<int32_t>& hs, const std::vector<int32_t>& gb) {
      const uint64_t n = hs.size();
      std::unique_ptr<Transfer> x = make_kv_transfer(dir, piece, ppb, base, base, dev, false, hs.data(), gb.data(), n, h.cfg());
      x->pool_launch = true;
      if (!dev) set_pool_table(x.get(), base, hs.data(), gb.data(), n);
      h.submit(std::move(x), n * slot_bytes, st, &kv);
    };
    for (int n : {1, 7, 300, 600}) {
      std::vector<int32_t> hs(n), gb(n);
      for (int i = 0; i < n; ++i) {
        hs[i] = (7 * i + 3) % static_cast<int>(slots);
        gb[i] = (11 * i + 1) % static_cast<int>(nb);
      }
      for (int rep = 0; rep < 3; ++rep) launch(MMA_H2D, hs, gb);  // queued back to back
      st.synchronize();
      CHECK(h.sync(), "sync");
      bool ok = true;
      for (int i = 0; i < n; ++i)
        for (uint32_t l = 0; l < L; ++l)
          for (uint32_t k = 0; k < 2; ++k)
            ok &= std::memcmp(layers[l].data() + (k * nb + gb[i]) * piece,
                              pool.data() + hs[i] * slot_bytes + (2 * l + k) * piece, piece) == 0;
      CHECK(ok, "pool fetch of %d blocks differs", n);
      // offload the fetched blocks back into other slots
      std::vector<int32_t> dest(n);
      for (int i = 0; i < n; ++i) dest[i] = (hs[i] + 1) % static_cast<int>(slots);
      auto want = pool;
      for (int j = 0; j < n; ++j)
        for (uint32_t l = 0; l < L; ++l)
          for (uint32_t k = 0; k < 2; ++k)
            std::memcpy(want.data() + dest[j] * slot_bytes + (2 * l + k) * piece,
                        layers[l].data() + (k * nb + gb[j]) * piece, piece);
      launch(MMA_D2H, dest, gb);
      st.synchronize();
      CHECK(h.sync(), "sync");
      CHECK(pool == want, "pool offload of %d blocks: pool differs", n);
    }
    CHECK(h.stats().sdma_commands.load() == cmds, "a pool launch used a copy engine");
  }
  {
    // Arena room: 16-byte pieces, one layer. A takes all but one segment, C
    // the last one, so B finds no room and goes through a record and the ring.
    FakeStream st;
    const uint64_t piece = 16, slot_bytes = 2 * piece;
    const uint32_t na = (kPoolTabEntries / kPoolTabSeg - 1) * kPoolTabSeg, nc = kPoolTabSeg, nbb = 3;
    const uint32_t total = na + nc + nbb;
    std::vector<uint8_t> pool = random_bytes(static_cast<uint64_t>(total) * slot_bytes, 62);
    std::vector<uint8_t> layer(2ull * total * piece, 0xA5);
    KvGeom kv;
    kv.piece = piece;
    kv.kstride = piece * total;
    kv.layers = 1;
    kv.layer_ptr[0] = reinterpret_cast<uint64_t>(layer.data());
    std::vector<int32_t> hs(total), gb(total);
    for (uint32_t i = 0; i < total; ++i) {
      hs[i] = static_cast<int32_t>((i * 7919ull) % total);  // 7919 is prime and does not divide total
      gb[i] = static_cast<int32_t>(total - 1 - i);
    }
    std::promise<void> gate;
    std::shared_future<void> open = gate.get_future().share();
    st.launch([open] { open.wait(); });  // holds the stream
    const uint32_t first[3] = {0, na, na + nc}, count[3] = {na, nc, nbb};
    bool launched[3];
    for (int t = 0; t < 3; ++t) {
      std::unique_ptr<Transfer> x = make_kv_transfer(MMA_H2D, piece, 2, reinterpret_cast<uint64_t>(pool.data()),
                                                     reinterpret_cast<uint64_t>(pool.data()), true, false,
                                                     hs.data() + first[t], gb.data() + first[t], count[t], h.cfg());
      x->pool_launch = true;
      Transfer* raw = x.get();
      h.submit(std::move(x), static_cast<uint64_t>(count[t]) * slot_bytes, st, &kv);
      launched[t] = raw->pool_launch;  // set by acquire; the held stream keeps the transfer alive
    }
    CHECK(launched[0] && launched[1] && !launched[2], "arena: expected launches A and C, ring for B (%d %d %d)",
          launched[0], launched[1], launched[2]);
    gate.set_value();
    st.synchronize();
    CHECK(h.sync(), "sync");
    bool ok = true;
    for (uint32_t i = 0; i < total; ++i)
      for (uint32_t k = 0; k < 2; ++k)
        ok &= std::memcmp(layer.data() + (k * total + gb[i]) * piece, pool.data() + hs[i] * slot_bytes + k * piece,
                          piece) == 0;
    CHECK(ok, "arena-bound pool fetches differ");
  }
  CHECK(h.stats().failed.load() == 0, "pool launches: failed transfers");
  std::printf("ok   pool launches in HBM and over the link; without arena room a transfer takes the ring\n");
}

// A deep queue of whole transfers on a stream that cannot progress yet: they
// take light slots, so submission does not wait for the stream (records alone
// would run out after 64), and every transfer lands once the stream runs.
void deep_queue_does_not_block() {
  Setup s;
  s.cfg = default_config();
  s.cfg.whole[0] = s.cfg.whole[1] = 4 * 1024 * 1024;
  Harness h(s);
  FakeStream st;
  std::promise<void> gate;
  std::shared_future<void> open = gate.get_future().share();
  st.launch([open] { open.wait(); });  // holds the stream
  const int n = 600;
  const uint64_t sz = 4096 + 16;
  auto src = random_bytes(sz * n, 8);
  std::vector<uint8_t> dst(sz * n, 0);
  auto submitted = std::async(std::launch::async, [&] {
    for (int i = 0; i < n; ++i)
      h.submit(linear(MMA_H2D, dst.data() + i * sz, src.data() + i * sz, sz, h.cfg()), sz, st);
  });
  const bool quick = submitted.wait_for(std::chrono::seconds(20)) == std::future_status::ready;
  CHECK(quick, "submitting %d whole transfers waited for the stream", n);
  gate.set_value();
  submitted.wait();
  st.synchronize();
  CHECK(h.sync(), "sync");
  CHECK(dst == src, "deep queue: bytes differ");
  CHECK(h.stats().failed.load() == 0, "deep queue: failed transfers");
  std::printf("ok   %d whole transfers queued behind a held stream without waiting for it\n", n);
}

// An early transfer whose dummy-task launch failed: the copy engines drain what
// they hold, the record is retired without a kernel, no sticky error is left,
// and the next transfer runs normally.
void unlaunched_transfer_drains() {
  Setup s;
  s.cfg = default_config();
  s.mask = MMA_PATH_CU | 0x3;
  Harness h(s);
  FakeStream st;
  const uint64_t n = 8 * 1024 * 1024;
  auto src = random_bytes(n, 5);
  std::vector<uint8_t> dst(n, 0);
  g_sticky.store(0);
  h.submit(linear(MMA_H2D, dst.data(), src.data(), n, h.cfg()), n, st, nullptr, true, false);
  CHECK(h.sync(), "an unlaunched transfer must be retired once its copy-engine commands drained");
  CHECK(g_sticky.load() == 0, "an unlaunched transfer must not leave a sticky error");
  CHECK(h.stats().failed.load() == 0 && h.stats().transfers.load() == 0, "unlaunched transfers are not counted");
  h.submit(linear(MMA_H2D, dst.data(), src.data(), n, h.cfg()), n, st, nullptr, true);
  st.synchronize();
  CHECK(h.sync(), "sync");
  CHECK(dst == src, "the transfer after an unlaunched one differs");
  std::printf("ok   an early transfer whose launch failed drains and retires without a sticky error\n");
}

void slow_engine_gets_fewer_tasks() {
  Setup s;
  s.cfg = default_config();
  s.cfg.merge = 1;
  s.engine_rates = {3000, 750};  // 4:1
  s.mask = 0x3;
  s.cmd_ns = 5000;
  Harness h(s);
  FakeStream st;
  const uint64_t n = 24 * 1024 * 1024;
  auto src = random_bytes(n, 3);
  std::vector<uint8_t> dst(n);
  h.submit(linear(MMA_H2D, dst.data(), src.data(), n, h.cfg()), n, st);
  st.synchronize();
  CHECK(h.sync(), "sync");
  CHECK(dst == src, "bytes differ");
  const double t0 = static_cast<double>(h.stats().path_tasks[0].load());
  const double t1 = static_cast<double>(h.stats().path_tasks[1].load());
  // 4:1 rates give about 3:1 on a quiet host; a loaded host's sleep overshoot narrows it.
  CHECK(t1 > 0 && t0 > 1.2 * t1, "fast engine %g tasks, slow engine %g tasks", t0, t1);
  std::printf("ok   a 4x slower copy engine pulls fewer micro-tasks: %g vs %g\n", t0, t1);
}

void submit_failures_rerouted() {
  Setup s;
  s.cfg = default_config();
  Harness h(s);
  FakeStream st;
  const uint64_t n = 4 * 1024 * 1024;
  auto src = random_bytes(n, 5);
  std::vector<uint8_t> dst(n);
  g_fault_submit_fail = 3;
  h.submit(linear(MMA_H2D, dst.data(), src.data(), n, h.cfg()), n, st);
  st.synchronize();
  CHECK(h.sync(), "sync");
  g_fault_submit_fail = 0;
  CHECK(dst == src, "bytes differ");
  CHECK(h.stats().submit_failures.load() >= 1 && h.stats().failed.load() == 0, "re-route");
  std::printf("ok   copy-engine submit failures re-routed to the CU path (%llu)\n",
              (unsigned long long)h.stats().submit_failures.load());
}

// Copy-engine commands refused during paged-KV transfers: a fetch's host->staging
// command (before anything moved) and an offload's staging->host command (after the
// CU gather into staging) both send their micro-tasks back to the CU path; the
// results are exact and no transfer fails.
void kv_submit_failures_rerouted() {
  Setup s;
  s.cfg = default_config();
  s.cfg.chunk = 8 * 1024;  // 4 pieces per micro-task
  s.mask = 0x3;            // copy engines only: every micro-task starts on an engine
  Harness h(s);
  FakeStream st;
  const uint32_t L = 2, ppb = 2 * L, slots = 16, nb = 20;
  const uint64_t piece = 2048, slot_bytes = piece * ppb;
  std::vector<uint8_t> pool = random_bytes(slots * slot_bytes, 21);
  std::vector<std::vector<uint8_t>> layers(L, std::vector<uint8_t>(2 * nb * piece, 0xA5));
  KvGeom kv;
  kv.piece = piece;
  kv.kstride = piece * nb;
  kv.layers = L;
  for (uint32_t l = 0; l < L; ++l) kv.layer_ptr[l] = reinterpret_cast<uint64_t>(layers[l].data());
  std::vector<int32_t> hs = {3, 7, 0, 12, 9, 15}, gb = {19, 2, 8, 5, 11, 0};
  const uint64_t host = reinterpret_cast<uint64_t>(pool.data());
  g_fault_submit_fail = 2;
  h.submit(make_kv_transfer(MMA_H2D, piece, ppb, host, host, false, true, hs.data(), gb.data(), hs.size(), h.cfg()),
           hs.size() * slot_bytes, st, &kv);
  st.synchronize();
  CHECK(h.sync(), "sync");
  bool ok = true;
  for (size_t i = 0; i < hs.size(); ++i)
    for (uint32_t l = 0; l < L; ++l)
      for (uint32_t k = 0; k < 2; ++k)
        ok &= std::memcmp(layers[l].data() + (k * nb + gb[i]) * piece,
                          pool.data() + hs[i] * slot_bytes + (2 * l + k) * piece, piece) == 0;
  CHECK(ok, "fetch with refused commands: pieces differ");
  const uint64_t after_fetch = h.stats().submit_failures.load();
  CHECK(after_fetch >= 1, "no refused command during the fetch");
  std::vector<int32_t> dest = {1, 2, 4, 5, 6, 8};
  auto want = pool;
  for (size_t j = 0; j < gb.size(); ++j)
    for (uint32_t l = 0; l < L; ++l)
      for (uint32_t k = 0; k < 2; ++k)
        std::memcpy(want.data() + dest[j] * slot_bytes + (2 * l + k) * piece,
                    layers[l].data() + (k * nb + gb[j]) * piece, piece);
  g_fault_submit_fail = 2;
  h.submit(make_kv_transfer(MMA_D2H, piece, ppb, host, host, false, true, dest.data(), gb.data(), gb.size(),
                            h.cfg()),
           gb.size() * slot_bytes, st, &kv);
  st.synchronize();
  CHECK(h.sync(), "sync");
  g_fault_submit_fail = 0;
  CHECK(pool == want, "offload with refused commands: pool differs");
  CHECK(h.stats().submit_failures.load() > after_fetch, "no refused command during the offload");
  CHECK(h.stats().failed.load() == 0 && g_sticky.load() == 0, "a refused command failed the transfer");
  std::printf("ok   refused copy-engine commands of KV fetch and offload re-routed to the CU path (%llu)\n",
              (unsigned long long)h.stats().submit_failures.load());
}

void two_streams_both_directions() {
  Setup s;
  s.cfg = default_config();
  Harness h(s);
  FakeStream a, b;
  const uint64_t n = 6 * 1024 * 1024 + 3;
  std::vector<std::vector<uint8_t>> srcs, dsts;
  for (int i = 0; i < 6; ++i) {
    srcs.push_back(random_bytes(n, 100 + i));
    dsts.emplace_back(n, 0);
  }
  for (int i = 0; i < 6; ++i) {
    FakeStream& st = i % 2 ? b : a;
    h.submit(linear(i % 2, dsts[i].data(), srcs[i].data(), n, h.cfg()), n, st);
  }
  a.synchronize();
  b.synchronize();
  CHECK(h.sync(), "sync");
  for (int i = 0; i < 6; ++i) CHECK(dsts[i] == srcs[i], "stream transfer %d differs", i);
  std::printf("ok   six transfers on two streams, both directions\n");
}

// ------------------------------------------------------------ device control
Setup device_setup() {
  Setup s;
  s.cfg = default_config();
  s.cfg.device = 1;
  s.cfg.device_cu_percent = 60;
  return s;
}

// Linear copies under device control, both directions: exact, every micro-task
// retired once; on an idle stream the copy engines carry their fixed share, on
// a stream with work pending none; the engine thread never runs.
void device_copies(bool idle) {
  Setup s = device_setup();
  Harness h(s);
  FakeStream st;
  for (int dir = 0; dir < 2; ++dir) {
    for (uint64_t n : {1ull, 777ull, 64ull * 1024, 300ull * 1024 + 5, 3ull * 1024 * 1024 + 123}) {
      auto src = random_bytes(n, static_cast<uint32_t>(n + 7 * dir));
      std::vector<uint8_t> dst(n + 64, 0xA5);
      auto x = linear(dir, dst.data() + 32, src.data(), n, h.cfg());
      const size_t tasks = x->tasks.size();
      const uint64_t before = sum_tasks(h.stats(), 0, MMA_NUM_PATHS);
      const uint64_t cmds = h.stats().sdma_commands.load();
      h.submit_device(std::move(x), n, st, nullptr, idle);
      st.synchronize();
      CHECK(h.sync(), "sync");
      CHECK(std::memcmp(dst.data() + 32, src.data(), n) == 0, "device dir=%d n=%llu idle=%d: bytes differ", dir,
            (unsigned long long)n, idle);
      CHECK(dst[31] == 0xA5 && dst[32 + n] == 0xA5, "device: bytes outside the destination changed");
      CHECK(sum_tasks(h.stats(), 0, MMA_NUM_PATHS) - before == tasks, "device: tasks retired");
      const uint64_t issued = h.stats().sdma_commands.load() - cmds;
      if (!idle) CHECK(issued == 0, "device: copy engines took part on a busy stream");
      if (idle && tasks >= 4) CHECK(issued >= 2, "device: the copy engines took no share (%llu commands)",
                                    (unsigned long long)issued);
    }
  }
  CHECK(h.stats().failed.load() == 0, "device: failed transfers");
  CHECK(h.stats().busy_ns.load() == 0, "device: the engine thread worked on a transfer");
  std::printf("ok   device control, %s stream: copies exact, cu tasks %llu, engine tasks %llu, no engine-thread work\n",
              idle ? "idle" : "busy", (unsigned long long)h.stats().path_tasks[MMA_NUM_PATHS - 1].load(),
              (unsigned long long)sum_tasks(h.stats(), 0, 16));
}

// Device control has no engine-thread phases, so a direction's duplex-only
// engines (here device-to-host engines 2-3) never take its copy-engine share:
// idle-stream copies in both directions use engines 0-1 alone.
void device_copies_keep_own_engines() {
  Setup s = device_setup();
  s.engine_rates = {2000, 2000, 2000, 2000};
  s.duplex[MMA_D2H] = 0xC;
  Harness h(s);
  FakeStream st;
  uint64_t init_bytes[4];  // each engine's warm-up command at init
  for (int e = 0; e < 4; ++e) init_bytes[e] = h.backend().engine_bytes(e);
  for (int dir = 0; dir < 2; ++dir) {
    const uint64_t n = 6ull * 1024 * 1024 + 9;
    auto src = random_bytes(n, static_cast<uint32_t>(31 + dir));
    std::vector<uint8_t> dst(n);
    h.submit_device(linear(dir, dst.data(), src.data(), n, h.cfg()), n, st, nullptr, true);
    st.synchronize();
    CHECK(h.sync(), "sync");
    CHECK(dst == src, "device dir=%d: bytes differ", dir);
  }
  const uint64_t e01 = h.backend().engine_bytes(0) + h.backend().engine_bytes(1) - init_bytes[0] - init_bytes[1];
  const uint64_t e23 = h.backend().engine_bytes(2) + h.backend().engine_bytes(3) - init_bytes[2] - init_bytes[3];
  CHECK(e01 > 0 && e23 == 0, "device control: engines 0-1 %llu bytes, duplex-only engines 2-3 %llu bytes",
        (unsigned long long)e01, (unsigned long long)e23);
  std::printf("ok   device control keeps to the direction's own engines (engines 0-1 %llu bytes, 2-3 none)\n",
              (unsigned long long)e01);
}

// Paged-KV fetch then offload under device control: the CU path alone.
void device_kv_roundtrip() {
  Setup s = device_setup();
  s.cfg.chunk = 8 * 1024;
  Harness h(s);
  FakeStream st;
  const uint32_t L = 3, ppb = 2 * L, slots = 24, nb = 30;
  const uint64_t piece = 2048, slot_bytes = piece * ppb;
  std::vector<uint8_t> pool = random_bytes(slots * slot_bytes, 41);
  std::vector<std::vector<uint8_t>> layers(L, std::vector<uint8_t>(2 * nb * piece, 0xA5));
  KvGeom kv;
  kv.piece = piece;
  kv.kstride = piece * nb;
  kv.layers = L;
  for (uint32_t l = 0; l < L; ++l) kv.layer_ptr[l] = reinterpret_cast<uint64_t>(layers[l].data());
  std::vector<int32_t> hs = {5, 0, 17, 3, 22, 9, 11}, gb = {2, 29, 7, 0, 13, 21, 4};
  const uint64_t host = reinterpret_cast<uint64_t>(pool.data());
  h.submit_device(make_kv_transfer(MMA_H2D, piece, ppb, host, host, false, true, hs.data(), gb.data(), hs.size(),
                                   h.cfg()),
                  hs.size() * slot_bytes, st, &kv, true);
  st.synchronize();
  CHECK(h.sync(), "sync");
  bool ok = true;
  for (size_t i = 0; i < hs.size(); ++i)
    for (uint32_t l = 0; l < L; ++l)
      for (uint32_t k = 0; k < 2; ++k)
        ok &= std::memcmp(layers[l].data() + (k * nb + gb[i]) * piece,
                          pool.data() + hs[i] * slot_bytes + (2 * l + k) * piece, piece) == 0;
  CHECK(ok, "device KV fetch: pieces differ");
  std::vector<int32_t> dest = {23, 2, 4, 6, 8, 10, 12};
  auto want = pool;
  for (size_t j = 0; j < gb.size(); ++j)
    for (uint32_t l = 0; l < L; ++l)
      for (uint32_t k = 0; k < 2; ++k)
        std::memcpy(want.data() + dest[j] * slot_bytes + (2 * l + k) * piece,
                    layers[l].data() + (k * nb + gb[j]) * piece, piece);
  h.submit_device(make_kv_transfer(MMA_D2H, piece, ppb, host, host, false, true, dest.data(), gb.data(), gb.size(),
                                   h.cfg()),
                  gb.size() * slot_bytes, st, &kv, true);
  st.synchronize();
  CHECK(h.sync(), "sync");
  CHECK(pool == want, "device KV offload: pool differs");
  CHECK(h.stats().sdma_commands.load() == 0, "device KV: a copy engine took part");
  CHECK(h.stats().failed.load() == 0 && h.stats().busy_ns.load() == 0, "device KV: failed or engine-thread work");
  std::printf("ok   device control: paged-KV fetch and offload exact on the CU path alone\n");
}

// More transfers than records, back to back on one stream: each submission
// recycles the records of retired transfers itself. Copy-engine commands that
// the runtime refuses go to the CU path. A transfer with more micro-tasks than
// a ring holds falls back to the engine thread.
void device_recycling_and_refusals() {
  Setup s = device_setup();
  Harness h(s);
  FakeStream st;
  const uint64_t n = 1024 * 1024 + 48;
  const int count = 3 * static_cast<int>(kRecords);
  auto src = random_bytes(n * count, 12);
  std::vector<uint8_t> dst(n * count, 0);
  for (int i = 0; i < count; ++i)
    h.submit_device(linear(i % 2, i % 2 ? src.data() + i * n : dst.data() + i * n,
                           i % 2 ? dst.data() + i * n : src.data() + i * n, n, h.cfg()),
                    n, st, nullptr, i % 3 != 0);
  st.synchronize();
  CHECK(h.sync(), "sync");
  for (int i = 0; i < count; ++i)
    CHECK(std::memcmp(dst.data() + i * n, src.data() + i * n, n) == 0, "device recycled transfer %d differs", i);
  CHECK(h.stats().transfers.load() == static_cast<uint64_t>(count), "device: %llu transfers retired",
        (unsigned long long)h.stats().transfers.load());
  // refused commands
  const uint64_t m = 6 * 1024 * 1024 + 9;
  auto src2 = random_bytes(m, 13);
  std::vector<uint8_t> dst2(m, 0);
  g_fault_submit_fail = 1;
  h.submit_device(linear(MMA_H2D, dst2.data(), src2.data(), m, h.cfg()), m, st, nullptr, true);
  st.synchronize();
  CHECK(h.sync(), "sync");
  g_fault_submit_fail = 0;
  CHECK(dst2 == src2, "device: refused command, bytes differ");
  CHECK(h.stats().submit_failures.load() == 1, "device: refused command not counted");
  CHECK(h.stats().failed.load() == 0 && g_sticky.load() == 0, "device: a refused command failed the transfer");
  CHECK(h.stats().busy_ns.load() == 0, "device: the engine thread worked on a transfer");
  // more micro-tasks than ring entries
  Setup s2 = device_setup();
  s2.cfg.chunk = 4 * 1024;
  s2.cfg.fallback = 8 * 1024;
  Harness h2(s2);
  const uint64_t big = (kRingSize + 3) * 4 * 1024ull + 5;
  auto src3 = random_bytes(big, 14);
  std::vector<uint8_t> dst3(big, 0);
  h2.submit_device(linear(MMA_H2D, dst3.data(), src3.data(), big, h2.cfg()), big, st, nullptr, true);
  st.synchronize();
  CHECK(h2.sync(), "sync");
  CHECK(dst3 == src3, "device fallback: bytes differ");
  CHECK(h2.stats().busy_ns.load() > 0, "device fallback: the engine thread did not take the transfer");
  std::printf("ok   device control: %d transfers recycle %u records, refused commands re-routed, "
              "a transfer beyond the ring falls back to the engine thread\n", count, kRecords);
}

// Device control with a launch that fails after the copy engines took their
// share: the call waits for them, frees the record, leaves no sticky error.
// Whole transfers in light slots are retired by later calls too.
void device_unlaunched_and_whole() {
  Setup s = device_setup();
  s.cfg.whole[0] = s.cfg.whole[1] = 1024 * 1024;
  Harness h(s);
  FakeStream st;
  const uint64_t n = 8 * 1024 * 1024;
  auto src = random_bytes(n, 15);
  std::vector<uint8_t> dst(n, 0);
  g_sticky.store(0);
  h.submit_device(linear(MMA_H2D, dst.data(), src.data(), n, h.cfg()), n, st, nullptr, true, false);
  CHECK(h.sync(), "sync after an unlaunched device transfer");
  CHECK(g_sticky.load() == 0 && h.stats().transfers.load() == 0, "unlaunched device transfer counted or sticky");
  h.submit_device(linear(MMA_H2D, dst.data(), src.data(), n, h.cfg()), n, st, nullptr, true);
  st.synchronize();
  CHECK(h.sync(), "sync");
  CHECK(dst == src, "device: transfer after an unlaunched one differs");
  // whole transfers behind a held stream
  std::promise<void> gate;
  std::shared_future<void> open = gate.get_future().share();
  st.launch([open] { open.wait(); });
  const int k = 300;
  const uint64_t sz = 20000;
  auto src2 = random_bytes(sz * k, 16);
  std::vector<uint8_t> dst2(sz * k, 0);
  auto submitted = std::async(std::launch::async, [&] {
    for (int i = 0; i < k; ++i)
      h.submit_device(linear(MMA_H2D, dst2.data() + i * sz, src2.data() + i * sz, sz, h.cfg()), sz, st, nullptr,
                      false);
  });
  CHECK(submitted.wait_for(std::chrono::seconds(20)) == std::future_status::ready,
        "device: whole transfers waited for the stream");
  gate.set_value();
  submitted.wait();
  st.synchronize();
  CHECK(h.sync(), "sync");
  CHECK(dst2 == src2, "device whole transfers differ");
  CHECK(h.stats().failed.load() == 0 && h.stats().busy_ns.load() == 0, "device whole: failed or engine-thread work");
  std::printf("ok   device control: a failed launch drains the copy engines; %d whole transfers retired by later calls\n",
              k);
}

// Shutting an engine down while a transfer is still in flight (process exit
// with a stream that has not reached the transfer): the memory the kernel
// shares with the engine stays allocated, and the kernel, once it runs, still
// finds its record and done tags.
void shutdown_in_flight_keeps_shared_memory() {
  Setup s;
  s.cfg = default_config();
  s.cfg.whole[0] = s.cfg.whole[1] = 4 * 1024 * 1024;
  Harness h(s);
  FakeStream st;
  std::promise<void> gate;
  std::shared_future<void> open = gate.get_future().share();
  st.launch([open] { open.wait(); });  // holds the stream
  const uint64_t n = 64 * 1024 + 7;
  auto src = random_bytes(n, 31);
  std::vector<uint8_t> dst(n, 0);
  h.submit(linear(MMA_H2D, dst.data(), src.data(), n, h.cfg()), n, st);
  Engine* e = h.engine(MMA_H2D);
  const bool idle = e->wait_idle(50);
  CHECK(!idle, "a transfer behind a held stream reported idle");
  const int frees = h.backend().frees();
  e->shutdown(idle);
  CHECK(h.backend().frees() == frees, "shared memory freed with a transfer in flight");
  gate.set_value();
  st.synchronize();
  CHECK(dst == src, "the transfer after an unreleased shutdown differs");
  std::printf("ok   shutdown with a transfer in flight keeps the memory its kernel uses\n");
}

// Pull-based selection against fixed splits decided at plan time, on two
// paths (the CU path and one copy engine) with a given rate ratio.
double timed_copy(double cu_rate, double eng_rate, uint32_t static_cu_percent, bool pull, uint64_t nap_ns = 0) {
  Setup s;
  s.cfg = default_config();
  s.cfg.nap_ns = nap_ns;  // naps sized for the fake paths' 1-2 GB/s, as in copies_are_exact
  s.cfg.overdue_gbs = nap_ns ? 1 : 0;
  s.cfg.cu_wgs = 1;
  s.cfg.merge = 1;
  s.cmd_ns = 0;
  s.engine_rates = {eng_rate};
  s.wave_rate = cu_rate / 4;  // 4 waves
  s.mask = MMA_PATH_CU | 0x1;
  if (!pull) {
    s.cfg.static_split = 1;
    s.cfg.static_cu_percent = static_cu_percent;
  }
  Harness h(s);
  FakeStream st;
  const uint64_t n = 32 * 1024 * 1024;
  std::vector<uint8_t> src(n, 1), dst(n);
  const auto t0 = std::chrono::steady_clock::now();
  h.submit(linear(MMA_H2D, dst.data(), src.data(), n, h.cfg()), n, st);
  st.synchronize();
  CHECK(h.sync(), "sync");
  const double ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
  CHECK(dst == src, "bytes differ");
  return ms;
}

// Another component's command on a copy engine: a path whose engine is in use
// while none of our commands is on it takes no work until the engine is free.
void foreign_work_skipped() {
  Setup s;
  s.cfg = default_config();
  s.engine_rates = {4000, 4000};
  s.cmd_ns = 5000;
  Harness h(s);
  FakeStream st;
  h.backend().foreign(0, 1500ull * 1000 * 1000);  // engine 0 busy for 1.5 s
  const uint64_t n = 8 * 1024 * 1024 + 7;
  auto src = random_bytes(n, 41);
  std::vector<uint8_t> dst(n);
  h.submit(linear(MMA_H2D, dst.data(), src.data(), n, h.cfg()), n, st);
  st.synchronize();
  CHECK(h.sync(), "sync");
  CHECK(dst == src, "bytes differ");
  CHECK(h.stats().foreign_skips.load() > 0, "engine 0 busy with foreign work was not skipped");
  CHECK(h.stats().path_tasks[0].load() == 0, "engine 0 took %llu micro-tasks while busy with foreign work",
        (unsigned long long)h.stats().path_tasks[0].load());
  std::printf("ok   a copy engine busy with foreign work is skipped (%llu skips; engine 1 %llu, CU %llu tasks)\n",
              (unsigned long long)h.stats().foreign_skips.load(), (unsigned long long)h.stats().path_tasks[1].load(),
              (unsigned long long)h.stats().path_tasks[16].load());
}

// Both directions on the same two copy engines, each engine running the
// commands of both from one in-order queue (Section 5.1.2, concurrent flows): a
// large host-to-device copy keeps merged 8 MiB commands queued on both engines
// while device-to-host copies (copy engines only) arrive one by one. The other
// direction's commands on an engine are neither foreign work (no skip) nor
// congestion: a device-to-host command waits for the 16 MiB queued before it,
// about four times the allowance for its own size, and within the allowance once
// those bytes count. Modelled engines at 2 GB/s, the overdue rule set for an
// 8 GB/s link, so that the host's memcpy stays inside the modelled times.
void duplex_peer_commands() {
  Setup s;
  s.cfg = default_config();
  s.cfg.chunk = 512 * 1024;
  s.cfg.fallback = 512 * 1024;
  s.cfg.merge = 16;  // commands up to 8 MiB
  s.cfg.overdue_gbs = 8;
  s.engine_rates = {2000, 2000};
  s.cmd_ns = 2000;
  s.mask = MMA_PATH_CU | 0x3;
  s.mask_d2h = 0x3;
  Harness h(s);
  FakeStream a, b;
  const uint64_t n = 192ull * 1024 * 1024 + 3, m = 1536 * 1024 + 5;
  const int k = 16;
  auto src = random_bytes(n, 51);
  std::vector<uint8_t> dst(n);
  std::vector<std::vector<uint8_t>> dsrc, ddst;
  for (int i = 0; i < k; ++i) {
    dsrc.push_back(random_bytes(m, 60 + i));
    ddst.emplace_back(m, 0);
  }
  h.submit(linear(MMA_H2D, dst.data(), src.data(), n, h.cfg()), n, a);
  sleep_ns(5000000);  // its commands are on both engines
  for (int i = 0; i < k; ++i) {  // arriving one by one while the large copy runs
    h.submit(linear(MMA_D2H, ddst[i].data(), dsrc[i].data(), m, h.cfg()), m, b);
    sleep_ns(1000000);
  }
  a.synchronize();
  b.synchronize();
  CHECK(h.sync(), "sync");
  CHECK(dst == src, "host-to-device bytes differ");
  for (int i = 0; i < k; ++i) CHECK(ddst[i] == dsrc[i], "device-to-host copy %d differs", i);
  const uint64_t skips = h.stats().foreign_skips.load(), backoffs = h.stats().congestion_backoffs.load();
  std::printf("     duplex: foreign skips %llu, congestion back-offs %llu\n", (unsigned long long)skips,
              (unsigned long long)backoffs);
  CHECK(skips == 0, "the other direction's commands counted as foreign work (%llu skips)",
        (unsigned long long)skips);
  CHECK(backoffs <= 1, "the other direction's commands counted as congestion (%llu back-offs; about 8 when they are)",
        (unsigned long long)backoffs);
  std::printf("ok   the other direction's commands on a shared copy engine are neither foreign work nor congestion\n");
}

// While the other direction moves, a direction pulls only from its duplex
// paths: here host-to-device engines 0-1 without the CU path, device-to-host
// engines 2-3 without the CU path. A device-to-host list issued while a long
// host-to-device copy runs takes engines 2-3 only, except for its small tensor,
// which only the CU path may carry; once the host-to-device copy is done, a
// second list uses its own paths again (engines 0-1 and the CU path). Exact in
// both directions.
void duplex_paths() {
  Setup s;
  s.cfg = default_config();
  s.cfg.chunk = 512 * 1024;
  s.cfg.fallback = 512 * 1024;
  s.cfg.merge = 16;
  s.engine_rates = {2000, 2000, 2000, 2000};
  s.cmd_ns = 2000;
  s.duplex[MMA_H2D] = 0x3;
  s.duplex[MMA_D2H] = 0xC;
  // A long hold: a loaded host (or a sanitizer build) may leave the
  // host-to-device engine thread unscheduled for more than the default 1 ms.
  s.cfg.duplex_hold_ns = 300000000;
  Harness h(s);
  FakeStream a, b;
  const uint64_t n = 160ull * 1024 * 1024 + 3;
  const std::vector<uint64_t> sizes = {8ull * 1024 * 1024 + 5, 4096, 4ull * 1024 * 1024};  // 4 KiB < small
  auto src = random_bytes(n, 71);
  std::vector<uint8_t> dst(n);
  std::vector<std::vector<uint8_t>> lsrc, ldst;
  for (int rep = 0; rep < 2; ++rep)
    for (size_t i = 0; i < sizes.size(); ++i) {
      lsrc.push_back(random_bytes(sizes[i], 80 + 10 * rep + static_cast<uint32_t>(i)));
      ldst.emplace_back(sizes[i], 0);
    }
  auto list = [&](int rep) {
    std::vector<mma_copy_desc_t> d;
    std::vector<uint64_t> z, sa, da;
    for (size_t i = 0; i < sizes.size(); ++i) {
      const size_t j = rep * sizes.size() + i;
      d.push_back({ldst[j].data(), lsrc[j].data(), sizes[i]});
      z.push_back(sizes[i]);
      sa.push_back(reinterpret_cast<uint64_t>(lsrc[j].data()));
      da.push_back(reinterpret_cast<uint64_t>(ldst[j].data()));
    }
    return make_list_transfer(MMA_D2H, d.data(), d.size(), z.data(), sa.data(), da.data(), h.cfg());
  };
  uint64_t total = 0;
  for (uint64_t z : sizes) total += z;
  auto d2h_tasks = [&]() {
    std::array<uint64_t, MMA_NUM_PATHS> t{};
    std::lock_guard<std::mutex> g(g_trace_mu);
    for (const auto& r : g_trace_buf)
      if (r.dir == MMA_D2H)
        for (int i = 0; i < MMA_NUM_PATHS; ++i) t[i] += r.path_tasks[i];
    g_trace_buf.clear();
    return t;
  };
  g_trace = 1;
  h.submit(linear(MMA_H2D, dst.data(), src.data(), n, h.cfg()), n, a);
  // the fake stream starts the transfer on a host thread: wait for it (a loaded host,
  // or a sanitizer build, can take several milliseconds)
  for (int i = 0; i < 2000 && !h.engine(MMA_H2D)->moving(); ++i) sleep_ns(1000000);
  CHECK(h.engine(MMA_H2D)->moving(), "the host-to-device copy is not moving after 2 s");
  h.submit(list(0), total, b);
  b.synchronize();
  CHECK(h.engine(MMA_D2H)->wait_idle(60000), "device-to-host list did not retire");
  const bool h2d_still_moving = h.engine(MMA_H2D)->moving();
  const auto t0 = d2h_tasks();
  a.synchronize();
  CHECK(h.sync(), "sync");
  sleep_ns(350000000);  // past the hold time
  h.submit(list(1), total, b);
  b.synchronize();
  CHECK(h.sync(), "sync");
  const auto t1 = d2h_tasks();
  g_trace = 0;
  CHECK(dst == src, "host-to-device bytes differ");
  for (size_t j = 0; j < ldst.size(); ++j) CHECK(ldst[j] == lsrc[j], "device-to-host tensor %zu differs", j);
  std::printf("     during: engines 0-1 %llu, 2-3 %llu, CU %llu tasks; after: engines 0-1 %llu, 2-3 %llu, CU %llu\n",
              (unsigned long long)(t0[0] + t0[1]), (unsigned long long)(t0[2] + t0[3]), (unsigned long long)t0[16],
              (unsigned long long)(t1[0] + t1[1]), (unsigned long long)(t1[2] + t1[3]), (unsigned long long)t1[16]);
  CHECK(h2d_still_moving, "the host-to-device copy ended before the device-to-host list (slow host?)");
  CHECK(t0[0] + t0[1] == 0 && t0[2] + t0[3] > 0 && t0[16] == 1,
        "while host-to-device moved: device-to-host tasks outside engines 2-3 and the small tensor's CU task");
  CHECK(t1[2] + t1[3] == 0 && t1[0] + t1[1] + t1[16] > 0, "alone: device-to-host tasks on engines 2-3");
  CHECK(h.stats().failed.load() == 0, "failed transfers");
  std::printf("ok   while the other direction moves, a direction pulls from its duplex paths only\n");
}

// Both directions at once with a launch over the link above the whole-transfer limit: it
// moves, for the other direction, from its start to its end, and a fetch is none while
// the engine thread moves the other direction (set_peer).
void link_launch_and_duplex_paths() {
  const uint32_t L = 1, ppb = 2, slots = 2100;
  const uint64_t piece = 1024, slot_bytes = piece * ppb;
  std::vector<uint8_t> pool = random_bytes(slots * slot_bytes, 91), layer(2 * slots * piece, 0xA5);
  KvGeom kv;
  kv.piece = piece;
  kv.kstride = piece * slots;
  kv.layers = L;
  kv.layer_ptr[0] = reinterpret_cast<uint64_t>(layer.data());
  const uint64_t base = reinterpret_cast<uint64_t>(pool.data());
  std::vector<int32_t> ids(slots);
  for (uint32_t i = 0; i < slots; ++i) ids[i] = static_cast<int32_t>(i);
  const uint64_t n = 24ull * 1024 * 1024 + 3;
  const auto src = random_bytes(n, 92);
  std::vector<uint8_t> dst(n);
  Setup s;
  s.cfg = default_config();
  s.cfg.cu_wgs = 16;
  s.cfg.whole[0] = s.cfg.whole[1] = 2 * MiB;
  s.duplex[MMA_H2D] = s.duplex[MMA_D2H] = 0x3;
  s.cfg.duplex_hold_ns = 10000000000;  // nothing here waits for its end
  for (const int dir : {MMA_H2D, MMA_D2H}) {
    Harness h(s);
    FakeStream a, b;
    const auto link = [&](int d) {
      std::unique_ptr<Transfer> x = make_kv_transfer(d, piece, ppb, base, base, false, true, ids.data(), ids.data(), slots, h.cfg());
      x->pool_launch = h.engine(d)->link_eligible(x.get(), kv, slots * slot_bytes, slot_bytes);
      set_pool_table(x.get(), base, ids.data(), ids.data(), slots);
      return x;
    };
    const int other = dir == MMA_H2D ? MMA_D2H : MMA_H2D;
    const auto cu_bytes = [&] { return h.stats().path_bytes[MMA_NUM_PATHS - 1].load(); };
    // queued behind other work the launch does not move yet
    std::promise<void> gate;
    std::shared_future<void> open = gate.get_future().share();
    a.launch([open] { open.wait(); });
    g_hold_links = true;
    std::unique_ptr<Transfer> x = link(dir);
    CHECK(x->pool_launch, "no launch over the link with the other direction idle");
    h.submit(std::move(x), slots * slot_bytes, a, &kv);
    CHECK(!h.engine(dir)->link_moving(), "a launch that has not started moves");
    gate.set_value();
    for (int i = 0; i < 2000 && !h.engine(dir)->link_moving(); ++i) sleep_ns(1000000);
    CHECK(h.engine(dir)->link_moving(), "a launch that has started does not move");
    // a copy of the other direction keeps to its duplex paths
    uint64_t before = cu_bytes();
    h.submit(linear(other, dst.data(), src.data(), n, h.cfg()), n, b);
    b.synchronize();
    CHECK(h.engine(other)->wait_idle(60000), "the copy did not retire");
    CHECK(h.engine(dir)->link_moving() && cu_bytes() == before, "beside the launch the CU path carried %llu bytes of the copy",
          static_cast<unsigned long long>(cu_bytes() - before));
    g_hold_links = false;
    a.synchronize();
    CHECK(!h.engine(dir)->link_moving(), "a launch that has ended moves");
    CHECK(h.sync(), "sync");
    before = cu_bytes();
    h.submit(linear(other, dst.data(), src.data(), n, h.cfg()), n, b);
    b.synchronize();
    CHECK(h.sync() && cu_bytes() > before && dst == src, "alone the copy uses the CU path, too");
    // the other direction moved less than the hold time ago, on this stream or another one
    CHECK(link(dir)->pool_launch, "no launch over the link behind a copy on its own stream");
    x = make_kv_transfer(dir, piece, ppb, base, base, false, true, ids.data(), ids.data(), slots, h.cfg());
    x->stream = &h;
    x->pool_launch = h.engine(dir)->link_eligible(x.get(), kv, slots * slot_bytes, slot_bytes);
    CHECK(x->pool_launch == (dir == MMA_D2H), "dir %d: launch over the link while the engine thread moves the other one: %d", dir,
          x->pool_launch);
    CHECK(h.stats().failed.load() == 0, "failed transfers");
  }
  {
    s.cfg.duplex_given[MMA_D2H] = true;  // chosen by the caller
    Harness h(s);
    FakeStream b;
    h.submit(linear(MMA_H2D, dst.data(), src.data(), n, h.cfg()), n, b);
    b.synchronize();
    std::unique_ptr<Transfer> x = make_kv_transfer(MMA_D2H, piece, ppb, base, base, false, true, ids.data(), ids.data(), slots, h.cfg());
    x->stream = &h;
    CHECK(!h.engine(MMA_D2H)->link_eligible(x.get(), kv, slots * slot_bytes, slot_bytes), "given duplex paths are not kept to");
    CHECK(h.sync(), "sync");
  }
  std::printf("ok   a large launch over the link moves for the other direction, and a fetch steps back for it\n");
}

void pull_tracks_best_static_split() {
  for (double ratio : {1.0, 2.0}) {
    const double eng = 1000, cu = 1000 * ratio;  // CU path ratio x faster
    double best = 1e30;
    std::printf("     rate ratio CU:SDMA = %g:1 -- static", ratio);
    // best of five runs each: the fake paths are host threads that sleep
    auto best_of5 = [&](uint32_t pct, bool pull, uint64_t nap_ns = 0) {
      double t = 1e30;
      for (int r = 0; r < 5; ++r) t = std::min(t, timed_copy(cu, eng, pct, pull, nap_ns));
      return t;
    };
    for (uint32_t pct : {0u, 33u, 50u, 67u, 100u}) {
      const double t = best_of5(pct, false);
      best = std::min(best, t);
      std::printf(" %u%%=%.1fms", pct, t);
    }
    const double p = best_of5(0, true);
    const double pn = best_of5(0, true, 50000);  // the engine thread napping between rounds
    std::printf(" | pull=%.1fms, with naps %.1fms\n", p, pn);
    // Quiet machines give pull <= best static (0.92-1.02 here); 5% allows for a busy host.
    CHECK(p <= best * 1.05, "pull %.1f ms vs best static %.1f ms at ratio %g", p, best, ratio);
    CHECK(pn <= best * 1.05, "pull with naps %.1f ms vs best static %.1f ms at ratio %g", pn, best, ratio);
    std::printf("     pull / best static = %.3f, with naps %.3f\n", p / best, pn / best);
  }
  std::printf("ok   pull-based selection tracks the best fixed split at 1:1 and 2:1, with and without naps\n");
}

}  // namespace

int main(int argc, char** argv) {
  const bool timing = !(argc > 1 && std::strcmp(argv[1], "--no-timing") == 0);
  const bool only_timing = argc > 1 && std::strcmp(argv[1], "--timing-only") == 0;
  if (!only_timing) {
    copies_are_exact(MMA_PATH_CU | 0x3, "CU + 2 engines");
    copies_are_exact(0x3, "2 engines");
    copies_are_exact(MMA_PATH_CU, "CU only");
    list_with_merging();
    kv_roundtrip(MMA_PATH_CU | 0x3, "CU + 2 engines, staging");
    kv_roundtrip(MMA_PATH_CU, "CU only");
    copies_are_exact(MMA_PATH_CU | 0x3, "CU + 2 engines, idle-stream early start", true);
    copies_are_exact(0x3, "2 engines, idle-stream early start", true);
    kv_roundtrip(MMA_PATH_CU | 0x3, "CU + 2 engines, staging, idle-stream early start", true);
    copies_are_exact(MMA_PATH_CU | 0x3, "CU + 2 engines, engine naps", false, 50000);
    copies_are_exact(0x3, "2 engines, engine naps", false, 50000);
    kv_roundtrip(MMA_PATH_CU | 0x3, "CU + 2 engines, staging, engine naps", false, 50000);
    unlaunched_transfer_drains();
    whole_transfers_on_cu();
    whole_kv_transfers();
    link_routes("few workgroups", kFewWorkgroups);
    link_routes("a few large pieces", kFewLarge);
    link_routes("chunk sizes", kChunks);
    hbm_pool_launches();
    deep_queue_does_not_block();
    submit_failures_rerouted();
    kv_submit_failures_rerouted();
    two_streams_both_directions();
    device_copies(true);
    device_copies(false);
    device_copies_keep_own_engines();
    device_kv_roundtrip();
    device_recycling_and_refusals();
    device_unlaunched_and_whole();
    shutdown_in_flight_keeps_shared_memory();
    foreign_work_skipped();
    duplex_paths();
    link_launch_and_duplex_paths();
  }
  if (timing) {
    duplex_peer_commands();
    slow_engine_gets_fewer_tasks();
    pull_tracks_best_static_split();
  }
  if (g_failures) {
    std::printf("FAILED: %d check(s)\n", g_failures);
    return 1;
  }
  std::printf("ALL OK\n");
  return 0;
}
