// How the workgroups of a block chain (one per tile, one launch for all blocks of a transform)
// wait for each other.  A chain needs all of them on the device at once, and whether they are is
// not the launch's to decide: a kernel on another stream or of another process may hold the
// place of some, the chain of another stream may hold its part and wait for the rest, or the free
// registers and LDS of a CU may lie in pieces.  So a launch first makes sure:
//   - every workgroup counts itself in (chain_arrive) and runs block 0, which waits for nobody;
//   - before block 1 it looks at the counts: all there, the chain goes on; after a bounded wait for
//     the rest, a workgroup seals the counts that are not complete (chain_decide).  A count only
//     grows, is complete or sealed for good, and a seal is a compare-and-swap on the same word, so
//     every workgroup comes to the same decision: one sealed count, and the launch is sealed.
//   - Sealed, the k workgroups counted so far run all blocks from the start, one block of the
//     whole frame at a time, tiles dealt out among them, with a barrier of those k after each
//     (chain_meet); they are all running, so that ends.  Workgroups that start later leave at
//     once.
// One count for all is a contended word (at 510 workgroups 3.5 us until the last has its
// answer, at 104 1.5); there are kChainGroups, a tile counts in one by its index.
// Progress words (flags, one per tile) hold a running count: a launch adds kChainStep to every
// word, whichever way it goes, so all words are equal between launches and a launch reads its
// base from its own tile's word; comparisons are of differences, so the count may wrap.  A launch
// uses one of two slots, the next one the other; it clears the one it does not use.
// The memory operations are a policy class: the device's in dc_chain.hpp, another one for a test on the host.
#pragma once
#include <stdint.h>

namespace nc {

constexpr uint32_t kChainStep = 16;  // at least the blocks of a launch

constexpr int kChainGroups = 8;

struct ChainSlot {
  struct alignas(128) Line {
    uint32_t v;
  };
  Line arrived[kChainGroups];  // workgroups that have started; sealed: bit 31, in bits 16 .. 30 how many of them go on
  Line ids;                    // numbers given to the workgroups of a sealed launch
  Line met;                    // arrivals at its barriers
};
constexpr int kChainWords = kChainGroups + 2;  // of a slot, each on a line of its own
static_assert(sizeof(ChainSlot) == 128 * kChainWords, "lines");

// The slot of a launch whose progress words start at base.
__host__ __device__ inline int chain_slot(uint32_t base) { return (base / kChainStep) & 1; }
// Tiles of n that count in group g.
__host__ __device__ inline uint32_t chain_group(uint32_t n, uint32_t g) { return (n + kChainGroups - 1 - g) / kChainGroups; }

// Word i of the slot that this launch does not use; all of them, by one workgroup of it.
template <class M>
__device__ inline void chain_clear(ChainSlot* slots, uint32_t base, int i) {
  M::store(&slots[1 - chain_slot(base)].arrived[0].v + i * (sizeof(ChainSlot::Line) / 4), 0u);
}

// One thread, before the workgroup stores anything: counts it in.  The result tells chain_late.
template <class M>
__device__ inline uint32_t chain_arrive(ChainSlot* slot, int tile) {
  return M::add(&slot->arrived[tile % kChainGroups].v, 1u);
}
// The workgroup started after its count was sealed: it must not store anything.
__host__ __device__ inline bool chain_late(uint32_t arrived_before) { return arrived_before >> 31; }

// Whether all n workgroups are running.  Waits at most `limit` polls for the rest; limit < 0 seals at
// once, and the answer is no whoever is there.
template <class M>
__device__ inline bool chain_decide(ChainSlot* slot, uint32_t n, int limit) {
  for (int spin = 0; spin < limit; ++spin) {
    bool complete = true, sealed = false;
    for (int g = 0; g < kChainGroups; ++g) {
      const uint32_t v = M::load(&slot->arrived[g].v);
      sealed |= v >> 31;
      complete &= v == chain_group(n, g);
    }
    if (complete) return true;
    if (sealed) break;
    M::pause();
  }
  bool sealed = limit < 0;
  for (int g = 0; g < kChainGroups; ++g)  // every count complete or sealed
    for (;;) {
      const uint32_t v = M::load(&slot->arrived[g].v);
      if (v == chain_group(n, g)) break;
      if (v >> 31 || M::cas(&slot->arrived[g].v, v, v | v << 16 | 1u << 31)) {
        sealed = true;
        break;
      }
    }
  return !sealed;
}

// The workgroups that go on with a sealed launch.
template <class M>
__device__ inline uint32_t chain_counted(ChainSlot* slot, uint32_t n) {
  uint32_t k = 0;
  for (int g = 0; g < kChainGroups; ++g) {
    const uint32_t v = M::load(&slot->arrived[g].v);
    k += v >> 31 ? v >> 16 & 0x7FFFu : chain_group(n, g);
  }
  return k;
}

// A tile's wait for a neighbour's word: true once it has published block b - 1.
__host__ __device__ inline bool chain_published(uint32_t flag, uint32_t base, int b) { return (int32_t)(flag - base) >= b; }

// One thread of each of the k workgroups of a sealed launch: the m-th barrier (m = 1, 2, ..).
// False if it gave up.
template <class M>
__device__ inline bool chain_meet(ChainSlot* slot, uint32_t k, uint32_t m, int limit) {
  M::add(&slot->met.v, 1u);
  for (int spin = 0; M::load(&slot->met.v) < k * m; ++spin) {
    if (spin > limit) return false;
    M::pause();
  }
  return true;
}

}  // namespace nc
