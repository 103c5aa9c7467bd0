// The block chains' protocol (csrc/chain_sync.hpp) on host threads: workgroups are threads, the
// device is a number of places, memory is atomics.  A "block" sets every tile of a row to a function
// of itself and its two neighbours.  Prints "ok <sealed launches>" or what went wrong.
#define __device__
#define __host__
#include "chain_sync.hpp"

#include <atomic>
#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <memory>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

using namespace nc;

struct HostMem {
  static uint32_t load(const uint32_t* p) { return __atomic_load_n(p, __ATOMIC_SEQ_CST); }
  static void store(uint32_t* p, uint32_t v) { __atomic_store_n(p, v, __ATOMIC_SEQ_CST); }
  static uint32_t add(uint32_t* p, uint32_t v) { return __atomic_fetch_add(p, v, __ATOMIC_SEQ_CST); }
  static bool cas(uint32_t* p, uint32_t a, uint32_t b) {
    return __atomic_compare_exchange_n(p, &a, b, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST);
  }
  static void pause() { std::this_thread::yield(); }
};

struct Device {  // places for workgroups; a workgroup keeps its place until it ends
  std::mutex m;
  std::condition_variable cv;
  int free;
  explicit Device(int places) : free(places) {}
  void enter() {
    std::unique_lock<std::mutex> l(m);
    cv.wait(l, [&] { return free > 0; });
    --free;
  }
  void leave() {
    { std::lock_guard<std::mutex> l(m); ++free; }
    cv.notify_all();
  }
};

static uint32_t mix(uint32_t a, uint32_t b, uint32_t c, uint32_t k) { return (a * 3 + b * 5 + c * 7 + k) * 2654435761u; }

struct Context {
  int n;
  std::vector<uint32_t> flags, buf[3];
  ChainSlot slots[2] = {};
  int sealed = 0, gave_up = 0;
  Context(int n, uint32_t base) : n(n), flags(n, base) {
    for (auto& b : buf) b.assign(n, 0);
  }
};

static std::atomic<int> failures{0};

// One workgroup of a launch of nb blocks from buf[0]; block b writes buf[1 + b % 2] (the second
// half of the input's life: buf[0] is overwritten by no block, as by no transform's chain before block 1)
static void workgroup(Context& c, int t, int nb, int limit) {
  const int n = c.n;
  auto at = [&](std::vector<uint32_t>& v, int i) { return i < 0 || i >= n ? 0u : HostMem::load(&v[i]); };
  auto src = [&](int b) -> std::vector<uint32_t>& { return b == 0 ? c.buf[0] : c.buf[1 + (b - 1) % 2]; };
  auto dst = [&](int b) -> std::vector<uint32_t>& { return c.buf[1 + b % 2]; };
  const uint32_t base = HostMem::load(&c.flags[t]);
  ChainSlot* const slot = &c.slots[chain_slot(base)];
  if (t == 0)
    for (int i = 0; i < kChainWords; ++i) chain_clear<HostMem>(c.slots, base, i);
  const uint32_t before = chain_arrive<HostMem>(slot, t);
  uint32_t own = mix(at(src(0), t - 1), at(src(0), t), at(src(0), t + 1), 0);
  std::this_thread::yield();
  if (!chain_late(before)) {
    HostMem::store(&dst(0)[t], own);
    HostMem::store(&c.flags[t], base + 1);
    if (chain_decide<HostMem>(slot, (uint32_t)n, limit)) {
      for (int b = 1; b < nb; ++b) {
        for (int d = -1; d <= 1; d += 2)
          if (t + d >= 0 && t + d < n) {
            long spin = 0;
            while (!chain_published(HostMem::load(&c.flags[t + d]), base, b)) {
              HostMem::pause();
              if (++spin > 200000000L) { ++failures; break; }
            }
          }
        own = mix(at(src(b), t - 1), own, at(src(b), t + 1), b);
        HostMem::store(&dst(b)[t], own);
        if (b + 1 < nb) HostMem::store(&c.flags[t], base + b + 1);
      }
    } else {
      const uint32_t k = chain_counted<HostMem>(slot, (uint32_t)n);
      const uint32_t id = HostMem::add(&slot->ids.v, 1u);
      if (id >= k) ++failures;
      if (id == 0) ++c.sealed;
      if (!chain_meet<HostMem>(slot, k, 1, 1 << 28)) ++failures;
      for (int b = 0; b < nb; ++b) {
        for (int i = (int)id; i < n; i += (int)k)
          HostMem::store(&dst(b)[i], mix(at(src(b), i - 1), at(src(b), i), at(src(b), i + 1), b));
        if (!chain_meet<HostMem>(slot, k, b + 2, 1 << 28)) ++failures;
      }
    }
  }
  HostMem::store(&c.flags[t], base + kChainStep);
}

static void launch(Device& dev, Context& c, int nb, int limit) {
  std::vector<uint32_t> want = c.buf[0];
  for (int b = 0; b < nb; ++b) {
    std::vector<uint32_t> next(c.n);
    for (int i = 0; i < c.n; ++i) next[i] = mix(i ? want[i - 1] : 0, want[i], i + 1 < c.n ? want[i + 1] : 0, b);
    want = next;
  }
  std::vector<std::thread> ts;
  for (int t = 0; t < c.n; ++t)
    ts.emplace_back([&, t] {
      dev.enter();
      workgroup(c, t, nb, limit);
      dev.leave();
    });
  for (auto& t : ts) t.join();
  if (c.buf[1 + (nb - 1) % 2] != want) {
    std::printf("wrong result: n %d, nb %d, limit %d\n", c.n, nb, limit);
    ++failures;
  }
  c.buf[0] = want;
  for (uint32_t f : c.flags)
    if (f != c.flags[0]) ++failures;
}

int main(int argc, char** argv) {
  const int places = std::atoi(argv[1]), n = std::atoi(argv[2]), other = std::atoi(argv[3]), limit = std::atoi(argv[4]);
  Device dev(places);
  // the progress words pass 2^31 and wrap on the way
  Context a(n, 0x7FFFFFC0u), b(other, 0xFFFFFFC0u);
  for (int i = 0; i < n; ++i) a.buf[0][i] = 17 * i + 1;
  for (int i = 0; i < other; ++i) b.buf[0][i] = 23 * i + 1;
  std::thread second([&] {
    if (other)
      for (int r = 0; r < 12; ++r) launch(dev, b, 2 + r % 15, limit);
  });
  for (int r = 0; r < 12; ++r) launch(dev, a, 2 + r % 15, limit);
  second.join();
  if (failures) return 1;
  std::printf("ok %d\n", a.sealed + b.sealed);
  return 0;
}
