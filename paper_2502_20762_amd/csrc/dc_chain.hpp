// Device side of the block chains, shared by the DC block kernels: the memory operations behind
// chain_sync.hpp, the exchange of edge pixels, and the steps of a launch that must wait.
#pragma once

#include "chain_sync.hpp"
#include "common.hpp"
#include "internal.hpp"

namespace nc {

struct DevMem {
  static __device__ __forceinline__ uint32_t load(const uint32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  static __device__ __forceinline__ void store(uint32_t* p, uint32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  static __device__ __forceinline__ uint32_t add(uint32_t* p, uint32_t v) {
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  static __device__ __forceinline__ bool cas(uint32_t* p, uint32_t from, uint32_t to) {
    return __hip_atomic_compare_exchange_strong(p, &from, to, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  static __device__ __forceinline__ void pause() { __builtin_amdgcn_s_sleep(1); }
};

// Polls are memory round trips, about 1.5 us: a neighbour's block and the barriers of a sealed
// launch may take a second (every workgroup waited for is running), the rest of the launch is
// waited for about 1.5 ms, longer than the launches of a codec that may hold its places.
constexpr int kChainWait = 1 << 16, kChainMeet = 1 << 20, kChainRest = 1 << 10;

// What a workgroup of a chain launch knows of it.
struct ChainRun {
  uint32_t* flags;
  int* status;
  ChainSlot* slots;
  uint32_t base;    // the tile's progress word at the start (the same in every lane, in a vector register)
  uint32_t before;  // chain_arrive's result (thread 0)
  uint32_t seen;    // count lane % kChainGroups as last seen
  int n, nb, limit;  // tiles, blocks; chain_decide's limit
  __device__ __forceinline__ ChainSlot* slot() const {
    return slots + __builtin_amdgcn_readfirstlane(chain_slot(base));
  }
};

__device__ __forceinline__ ChainRun chain_begin(const DcChainArgs& ca, int tile, int n) {
  ChainRun r;
  r.flags = (uint32_t*)ca.flags;
  r.status = ca.status;
  r.slots = ca.slots;
  r.n = n;
  r.nb = ca.nb;
  r.limit = ca.seal ? -1 : kChainRest;
  r.base = DevMem::load(r.flags + tile);
  r.before = r.seen = 0;
  return r;
}

// Block 0 in three places.  Once the band is in, before the depthwise, which hides a
// part of the answer's way.
__device__ __forceinline__ void chain_count_in(ChainRun& r, int tile) {
  if (threadIdx.x == 0) r.before = chain_arrive<DevMem>(r.slot(), tile);
  if (tile == 0 && threadIdx.x < kChainWords) chain_clear<DevMem>(r.slots, r.base, threadIdx.x);
}
// Before a later barrier: the answer for every wave, through LDS.
__device__ __forceinline__ void chain_tell(const ChainRun& r, char* word) {
  if (threadIdx.x == 0) *(uint32_t*)word = r.before;
}
// Before the output: whether the workgroup is too late to store anything; the counts as they are now.
__device__ __forceinline__ bool chain_too_late(ChainRun& r, const char* word) {
  r.seen = DevMem::load(&r.slot()->arrived[threadIdx.x % kChainGroups].v);
  return chain_late((uint32_t)__builtin_amdgcn_readfirstlane(*(const int*)word));
}

// Block b is done and its edge pixels are in memory.  The last word of a launch is the next
// one's base.
__device__ __forceinline__ void chain_publish(const ChainRun& r, int tile, int b) {
  if (threadIdx.x == 0) DevMem::store(r.flags + tile, r.base + (b == r.nb - 2 ? kChainStep : (uint32_t)b + 1));
}
// The way out of a launch without publications.
__device__ __forceinline__ void chain_end(const ChainRun& r, int tile) {
  if (threadIdx.x == 0) DevMem::store(r.flags + tile, r.base + kChainStep);
}

// Whether the chain goes on past block 0, for a wave.  Every wave comes to the same answer.
__device__ __forceinline__ bool chain_goes_on(const ChainRun& r) {
  if (r.limit >= 0 && __ballot(r.seen != chain_group((uint32_t)r.n, threadIdx.x % kChainGroups)) == 0) return true;
  uint32_t go = 0;
  if ((threadIdx.x & 63) == 0) go = chain_decide<DevMem>(r.slot(), (uint32_t)r.n, r.limit) ? 1 : 0;
  return __builtin_amdgcn_readfirstlane((int)go) != 0;
}

// Wave 0 waits until every neighbouring tile has published block b - 1 (its edge
// pixels are in memory then): one lane per neighbour polls its word.
__device__ __forceinline__ void chain_wait(const ChainRun& r, int b, int lane, int tyi, int txi, int tiles_y, int tiles_x) {
  if (lane >= 9 || lane == 4) return;
  const int ny = tyi + lane / 3 - 1, nx = txi + lane % 3 - 1;
  if (ny < 0 || ny >= tiles_y || nx < 0 || nx >= tiles_x) return;
  const uint32_t* f = r.flags + ny * tiles_x + nx;
  for (int spin = 0; !chain_published(DevMem::load(f), r.base, b); ++spin) {
    if (spin > kChainWait) {  // give up, record it
      __hip_atomic_store(r.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      break;
    }
    DevMem::pause();
  }
}

// A barrier of the k workgroups of a sealed launch: what they stored before it is seen by all
// loads after it (the fences write back this XCD's L2 and drop its older lines).
__device__ __forceinline__ void chain_meet_all(const ChainRun& r, uint32_t k, uint32_t m) {
  __threadfence();
  __syncthreads();
  if (threadIdx.x == 0 && !chain_meet<DevMem>(r.slot(), k, m, kChainMeet))
    __hip_atomic_store(r.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  __threadfence();
}

// The rest of a sealed launch: run(b, t) computes block b of tile t whole, from memory to
// memory.  word: LDS that nobody uses at this point.
template <typename F>
__device__ __forceinline__ void chain_sealed(const ChainRun& r, int nb, uint32_t* word, F&& run) {
  const uint32_t k = (uint32_t)__builtin_amdgcn_readfirstlane((int)chain_counted<DevMem>(r.slot(), (uint32_t)r.n));
  if (threadIdx.x == 0) *word = DevMem::add(&r.slot()->ids.v, 1u);
  __syncthreads();
  const int id = __builtin_amdgcn_readfirstlane((int)*word);
  chain_meet_all(r, k, 1);  // the edge stores of everyone's block 0 are done
  for (int b = 0; b < nb; ++b) {
    for (int t = id; t < r.n; t += (int)k) {
      run(b, t);
      __syncthreads();
    }
    chain_meet_all(r, k, b + 2);
  }
}

// 16-byte device-coherent accesses (the sc1 policy of device-scope atomics:
// past this XCD's L2 to the device's point of coherence), whole 128-byte lines
// per 8 lanes, without a cache-wide fence (a fence would write back or drop
// the whole L2, weights included).
// N loads and the wait for them are one asm block, so nothing reads a result,
// or reuses a register of it, while a load is in flight.
template <int N, typename V, typename T>
__device__ __forceinline__ void load_coherent16(V (&v)[N], const T* const (&p)[N]) {
  static_assert(sizeof(V) == 16 && (N == 2 || N == 3 || N == 5 || N == 7), "ring loads per lane");
  if constexpr (N == 2)
    asm volatile(
        "global_load_dwordx4 %0, %2, off sc1\n\t"
        "global_load_dwordx4 %1, %3, off sc1\n\t"
        "s_waitcnt vmcnt(0)"
        : "=&v"(v[0]), "=&v"(v[1])
        : "v"(p[0]), "v"(p[1])
        : "memory");
  else if constexpr (N == 3)
    asm volatile(
        "global_load_dwordx4 %0, %3, off sc1\n\t"
        "global_load_dwordx4 %1, %4, off sc1\n\t"
        "global_load_dwordx4 %2, %5, off sc1\n\t"
        "s_waitcnt vmcnt(0)"
        : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2])
        : "v"(p[0]), "v"(p[1]), "v"(p[2])
        : "memory");
  else if constexpr (N == 5)
    asm volatile(
        "global_load_dwordx4 %0, %5, off sc1\n\t"
        "global_load_dwordx4 %1, %6, off sc1\n\t"
        "global_load_dwordx4 %2, %7, off sc1\n\t"
        "global_load_dwordx4 %3, %8, off sc1\n\t"
        "global_load_dwordx4 %4, %9, off sc1\n\t"
        "s_waitcnt vmcnt(0)"
        : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4])
        : "v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[3]), "v"(p[4])
        : "memory");
  else
    asm volatile(
        "global_load_dwordx4 %0, %7, off sc1\n\t"
        "global_load_dwordx4 %1, %8, off sc1\n\t"
        "global_load_dwordx4 %2, %9, off sc1\n\t"
        "global_load_dwordx4 %3, %10, off sc1\n\t"
        "global_load_dwordx4 %4, %11, off sc1\n\t"
        "global_load_dwordx4 %5, %12, off sc1\n\t"
        "global_load_dwordx4 %6, %13, off sc1\n\t"
        "s_waitcnt vmcnt(0)"
        : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6])
        : "v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[3]), "v"(p[4]), "v"(p[5]), "v"(p[6])
        : "memory");
}
// A store of more than 8 bytes still reads its data registers when the next instructions issue:
// two wait states must lie before a VALU instruction may write them.  The compiler keeps that
// distance for its own stores but does not see into this one.
template <typename V, typename T>
__device__ __forceinline__ void store_coherent16(T* p, V v) {
  static_assert(sizeof(V) == 16, "16 bytes");
  asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
}

}  // namespace nc
