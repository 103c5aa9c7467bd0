// Entropy coding of the quantised latent (Fig. 4 "AE" / "AD", Fig. 6): rANS
// (Duda 2013, range variant: 32-bit state in [2^16, 2^32), 16-bit words,
// M = 2^16) on quantised-scale Gaussian tables.
//
// A stream is 8192 symbols coded by the 64 lanes of one wave in lock step:
// symbol i of the stream belongs to lane i % 64 at step i / 64.  At every
// (step, sub-symbol) the lanes that move a word do so in lane order (ballot +
// popcount give each its slot), so a stream is one contiguous run of words.
// An escaped symbol (|q| beyond its table) continues with one 16-bit field
// of frequency 1: 32768 * sign + |q| - R - 1.
//
// Every coder kernel first stages what its sequential loop touches into LDS
// with direct global->LDS loads issued back to back and one wait (the tables,
// the stream's symbols and scale indices, the decoder also the stream's
// words), so the loop over the 128 steps never waits on global memory.
//
// k_rans_encode  one wave per stream of up to three containers: encodes backwards into
//                the stream's scratch slot, words ending at the slot's end
// k_rans_pack    one workgroup per stream: copies the words into its container; a
//                container's first workgroup writes the header and length table
// k_rans_decode  one wave per stream: checks the container, decodes forward,
//                every word read bounded by the stream's length; flags a
//                truncated or inconsistent stream instead of reading past it
#include <type_traits>

#include "common.hpp"
#include "internal.hpp"

namespace nc {

namespace {

constexpr uint32_t kRansL = 1u << 16;

// Direct global->LDS load of 4 bytes per lane: lane l's bytes land at
// lds_wave_base + 4 l.  Callers wait with s_waitcnt vmcnt before reading.
__device__ __forceinline__ void dma4(const void* g, const void* lds_wave_base) {
  const uint32_t m = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)lds_wave_base;
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" ::"v"(g), "s"(m) : "memory", "m0");
}

// Stages n16 16-byte chunks from g into LDS at lds (one wave, 1 KiB per load
// instruction).
__device__ __forceinline__ void stage16(const void* g, void* lds, int n16, int lane) {
  for (int i = 0; i < n16; i += 64)
    if (i + lane < n16) dma16((const uint8_t*)g + 16 * (i + lane), (uint8_t*)lds + 16 * i);
}

// Lanes below this one in a ballot mask.
__device__ __forceinline__ uint32_t below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += (uint32_t)__shfl_xor((int)v, off, 64);
  return v;
}

__device__ __forceinline__ uint32_t wave_or(uint32_t v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v |= (uint32_t)__shfl_xor((int)v, off, 64);
  return v;
}

}  // namespace

// The section of a launch's workgroup, and the stream of the section it takes.
__device__ __forceinline__ const RansSection& section_of(const RansSections& a, int& s) {
  int i = 0;
  while (i + 1 < a.count && s >= a.sec[i].ns) s -= a.sec[i++].ns;
  return a.sec[i];
}

// One wave (workgroup) per stream.  The table lookup of a step (symbol and
// scale index, then R and the scale's first start, then the entry) runs three
// steps ahead of the state chain, one stage per step, so none of its LDS reads
// is waited for on the chain; what depends on the entry alone (the shifted
// frequency, its reciprocal, the escape test) is formed there too.
//
// Bound by one wave's chain of 128 steps, so by its instructions: the quotient x / f
// (below 2^16) is estimated from below, trunc(x rcp(f) - 2^-5) (x rcp(f) is
// within 2^-6 of x / f), so it is q or q - 1 and one correction upwards makes the
// new state exact: (q << 16) + (x - q f) + c = x + c + q (2^16 - f).  All steps but a
// stream's last take every lane.  1080p (255 streams): 33.6 us before, 29.5 now,
// of which 5.4 stage the tables.
__global__ __launch_bounds__(64) void k_rans_encode(RansSections secs, const uint16_t* tab, uint16_t* scratch,
                                                  int64_t max_words, uint32_t* lens) {
  __shared__ __align__(16) uint16_t st[kTabEncU16];
  __shared__ __align__(16) int16_t sq[kRansStream];
  __shared__ __align__(16) uint8_t sk[kRansStream];
  const int lane = threadIdx.x;
  int s = blockIdx.x;
  const RansSection& sec = section_of(secs, s);
  const int64_t base = (int64_t)s * kRansStream;
  const int16_t* const q = sec.q + base;
  const uint8_t* const kidx = sec.k + base;
  const int cnt = (int)min((int64_t)kRansStream, sec.n - base);
  const int steps = (cnt + 63) / 64;
  stage16(tab, st, kTabEncU16 / 8, lane);
  const int nq = cnt / 8, nk = cnt / 16;  // whole 16-byte chunks; q and k are 16-byte aligned
  stage16(q, sq, nq, lane);
  stage16(kidx, sk, nk, lane);
  if (8 * nq + lane < cnt) sq[8 * nq + lane] = q[8 * nq + lane];
  if (16 * nk + lane < cnt) sk[16 * nk + lane] = kidx[16 * nk + lane];
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  const uint16_t* sst = st + kTabStarts;
  const uint2* shead = (const uint2*)st;  // scale j: (R | first << 16, ..)
  // positions past cnt read values that are never used; every index stays
  // inside the tables
  int aq = 0, ak = 0;           // stage A: symbol, scale index
  int bq = 0, bR = 0, bo = 0;   // stage B: symbol, R, first start
  uint32_t cc = 0, cf = 1;      // stage C: start, frequency,
  float crcp = 1.f;             //          its reciprocal,
  int cq = 0, cR = 0;           //          symbol, R
  bool cesc = false;            //          escaped
  uint32_t c0 = 0, c1 = 0;      // stage C's reads, used one step later
  int dq = 0, dR = 0;
  bool desc = false;
  auto stage_a = [&](int u) {
    if (u >= 0) {
      aq = sq[u * 64 + lane];
      ak = sk[u * 64 + lane];
    }
  };
  auto stage_b = [&]() {
    const uint32_t h = shead[min(ak, kCoderScales - 1)].x;
    bq = aq;
    bR = (int)(h & 0xFFFFu);
    bo = (int)(h >> 16);
  };
  auto stage_c = [&]() {
    desc = (uint32_t)(bq + bR) > (uint32_t)(2 * bR);
    const int i = bo + (desc ? 2 * bR + 1 : bq + bR);
    c0 = sst[i];
    c1 = sst[i + 1];
    dq = bq;
    dR = bR;
  };
  auto stage_d = [&]() {
    cc = c0;
    cf = (c1 - c0) & 0xFFFFu;
    crcp = __builtin_amdgcn_rcpf((float)cf);
    cq = dq;
    cR = dR;
    cesc = desc;
  };
  stage_a(steps - 1);
  stage_b();
  stage_c();
  stage_d();
  stage_a(steps - 2);
  stage_b();
  stage_c();
  stage_a(steps - 3);
  stage_b();
  stage_a(steps - 4);
  // words go to the end of the stream's slot, counted back from it
  uint16_t* const slot = scratch + (int64_t)blockIdx.x * max_words;
  uint32_t w = (uint32_t)max_words;  // first word written so far
  uint32_t x = kRansL;
  auto step = [&](int t, auto allc) __attribute__((always_inline)) {
    constexpr bool all = decltype(allc)::value;
    const bool act = all || t * 64 + lane < cnt;
    const uint32_t c = cc, f = act ? cf : 1u;
    const float rf = crcp;
    const int qv = cq, R = cR;
    const bool esc = act && cesc;
    stage_d();
    stage_c();
    stage_b();
    stage_a(t - 4);
    if (const uint64_t m = __ballot(esc)) {
      // the field follows the escape in decoding order, so it is coded first;
      // with frequency 1 every escaped state moves a word out
      w -= (uint32_t)__popcll(m);
      if (esc) {
        const uint32_t fld = (qv < 0 ? 32768u : 0u) + (uint32_t)(abs(qv) - R - 1);
        slot[w + below(m)] = (uint16_t)x;
        x = (x & 0xFFFF0000u) | fld;
      }
    }
    const bool emit = act && x >= (f << 16);
    const uint64_t m = __ballot(emit);
    w -= (uint32_t)__popcll(m);
    if (emit) slot[w + below(m)] = (uint16_t)x;
    x = emit ? x >> 16 : x;
    const uint32_t q0 = (uint32_t)fmaxf(fmaf((float)x, rf, -0.03125f), 0.f);
    const uint32_t r0 = x - __umul24(q0, f);
    const uint32_t y = x + c + __umul24(q0, 65536u - f) + (r0 >= f ? 65536u - f : 0u);
    x = act ? y : x;
  };
  if (steps > 0) step(steps - 1, std::false_type{});
  for (int t = steps - 2; t >= 0; --t) step(t, std::true_type{});
  // the 64 final states open the stream: lane l at words 2l (high) and 2l + 1
  w -= 128;
  slot[w + 2 * lane] = (uint16_t)(x >> 16);
  slot[w + 2 * lane + 1] = (uint16_t)(x & 0xFFFFu);
  if (lane == 0) lens[blockIdx.x] = (uint32_t)max_words - w;
}

// One workgroup per stream: the stream's place in its container is the sum of
// the lengths before it (every workgroup sums them itself, so no separate scan
// pass); a container's first workgroup also writes the header and the length table.
__global__ __launch_bounds__(256) void k_rans_pack(RansSections secs, const uint16_t* __restrict__ scratch,
                                                 int64_t max_words, const uint32_t* __restrict__ all_lens) {
  __shared__ uint32_t sa[4], stot[4];
  int s = blockIdx.x;
  const RansSection& sec = section_of(secs, s);
  const uint32_t* const lens = all_lens + (blockIdx.x - s);
  const int ns = sec.ns;
  uint8_t* const out = sec.out;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t a = 0, tot = 0;
  for (int i = threadIdx.x; i < ns; i += 256) {
    const uint32_t v = lens[i];
    tot += v;
    a += i < s ? v : 0u;
  }
  a = wave_sum(a);
  tot = wave_sum(tot);
  if (lane == 0) {
    sa[wave] = a;
    stot[wave] = tot;
  }
  __syncthreads();
  a = sa[0] + sa[1] + sa[2] + sa[3];
  tot = stot[0] + stot[1] + stot[2] + stot[3];
  const uint32_t len = lens[s];
  const uint16_t* src = scratch + (int64_t)(blockIdx.x + 1) * max_words - len;
  uint16_t* dst = (uint16_t*)(out + rans_payload_offset(ns)) + a;
  // eight loads in flight per thread (both ends lie at any word); one at a time took
  // 8.6 us at 1080p (255 streams), this 6.0
  uint32_t i = threadIdx.x;
  for (; i + 7 * 256 < len; i += 8 * 256) {
    uint16_t v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = src[i + 256 * e];
#pragma unroll
    for (int e = 0; e < 8; ++e) dst[i + 256 * e] = v[e];
  }
  for (; i < len; i += 256) dst[i] = src[i];
  if (s == 0) {
    uint16_t* ltab = (uint16_t*)(out + kRansHeader);
    for (int i = threadIdx.x; i < ns; i += 256) ltab[i] = (uint16_t)lens[i];
    if (threadIdx.x == 0) {
      uint32_t* h = (uint32_t*)out;
      h[0] = kRansMagic;
      h[1] = kRansVersion;
      h[2] = (uint32_t)sec.n;
      h[3] = (uint32_t)kRansStream;
      h[4] = (uint32_t)ns;
      if (ns & 1) ltab[ns] = 0;  // pad to 4 bytes
      *sec.nbytes = (uint64_t)rans_payload_offset(ns) + 2ull * tot;
    }
  }
}

// One wave (workgroup) per stream.  LDS holds the whole coder table block,
// the stream's scale indices and the stream's words (word i at sw[par + i],
// par the parity of the stream's start, so that whole dwords can be staged).
// Every workgroup checks the container header and sums the length table up to
// its stream itself.  Each writes its error bits to errs[s]; the last one to
// finish (a ticket on *count, which it resets) merges them into *status_out.
// Bound by the state chain's three dependent LDS reads per step (bucket, starts,
// word); only lanes that meet a run or a crowded bucket leave the straight path.
// 1080p (255 streams): 57 us before, 44.5 now, of which 7.6 stage the tables.
__global__ __launch_bounds__(64) void k_rans_decode(const uint8_t* in, uint64_t in_bytes, const uint8_t* kidx,
                                                  int64_t n, const uint16_t* tab, uint32_t* errs, uint32_t* count,
                                                  int16_t* q, int32_t* status_out) {
  __shared__ __align__(16) uint16_t st[kTabU16];
  __shared__ __align__(16) uint8_t sk[kRansStream];
  __shared__ __align__(16) uint16_t sw[kRansMaxWords + 4];
  const int lane = threadIdx.x;
  const int s = blockIdx.x;
  const int ns = (int)((n + kRansStream - 1) / kRansStream);
  const int64_t base = (int64_t)s * kRansStream;
  const int cnt = (int)min((int64_t)kRansStream, n - base);
  const int steps = (cnt + 63) / 64;
  stage16(tab, st, kTabU16 / 8, lane);
  const int nk = cnt / 16;  // k is 16-byte aligned
  stage16(kidx + base, sk, nk, lane);
  if (16 * nk + lane < cnt) sk[16 * nk + lane] = kidx[base + 16 * nk + lane];
  // container check (wave-uniform: every lane reads the same words; all loads
  // issued before the first use)
  bool bad = in_bytes < (uint64_t)rans_payload_offset(ns);
  const uint16_t* ltab = (const uint16_t*)(in + kRansHeader);
  uint32_t a = 0, tot = 0;
  if (!bad) {
    const uint32_t* h = (const uint32_t*)in;
    const uint32_t h0 = h[0], h1 = h[1], h2 = h[2], h3 = h[3], h4 = h[4];
#pragma unroll 4
    for (int i = lane; i < ns; i += 64) {
      const uint32_t v = ltab[i];
      tot += v;
      a += i < s ? v : 0u;
    }
    bad = (h0 != kRansMagic) | (h1 != kRansVersion) | (h2 != (uint32_t)n) | (h3 != (uint32_t)kRansStream) |
          (h4 != (uint32_t)ns);
  }
  // the sums are wave-uniform; readfirstlane puts them in scalar registers (the
  // LDS destination of the word staging below goes through M0)
  a = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_sum(a));
  tot = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_sum(tot));
  if (!bad && (uint64_t)rans_payload_offset(ns) + 2ull * tot > in_bytes) bad = true;
  uint32_t err = bad ? 1u : 0u;
  uint32_t len = bad ? 0u : (uint32_t)ltab[s];
  if (len > (uint32_t)kRansMaxWords) {
    err |= 2;
    len = 0;
  }
  if (len < 128) err |= 2;
  // the stream's words are u16 indices [g0, g1) of the container
  const uint64_t g0 = (uint64_t)(rans_payload_offset(ns) / 2) + a, g1 = g0 + len;
  const int par = (int)(g0 & 1);
  {
    // whole dwords d0 .. d1 - 1 inside [g0, g1); dword d lands at sw[2 (d - g0 / 2)]
    const uint64_t d0 = (g0 + 1) / 2, d1 = g1 / 2;
    const int nd = d1 > d0 ? (int)(d1 - d0) : 0;
    const uint32_t* src = (const uint32_t*)in + d0;
    uint16_t* dst = sw + 2 * (d0 - g0 / 2);
    for (int i = 0; i < nd; i += 64)
      if (i + lane < nd) dma4(src + i + lane, dst + 2 * i);
    const uint16_t* in16 = (const uint16_t*)in;
    if (lane == 0 && len > 0 && par) sw[1] = in16[g0];                          // odd first word
    if (lane == 1 && len > 0 && (g1 & 1)) sw[par + len - 1] = in16[g1 - 1];   // odd last word
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  const uint16_t* sst = st + kTabStarts;
  const uint16_t* sbk = st + kTabBuckets;
  // a word past the stream reads the zero after it; that it happened shows in the
  // final position
  if (lane == 2) sw[par + len] = 0;
  __syncthreads();
  auto word = [&](uint32_t i) -> uint32_t { return (uint32_t)sw[par + min(i, len)]; };
  uint32_t x = (word(2 * lane) << 16) | word(2 * lane + 1);
  uint32_t pos = 128;
  // lane-ordered renormalisation reads of the lanes in need
  auto refill = [&](bool need) __attribute__((always_inline)) {
    const uint64_t m = __ballot(need);
    const uint32_t v = (x << 16) | word(pos + below(m));
    x = need ? v : x;
    pos += (uint32_t)__popcll(m);
  };
  // table coordinates that do not depend on the state run ahead of the state
  // chain: the scale index two steps, its R, first start and tail counts one
  // step (positions past cnt read values that are never used; every index
  // stays inside the tables).  The index is clamped where it is used, not where
  // it is loaded, so that the load is not waited for until the next step.
  const uint2* shead = (const uint2*)st;  // scale j: (R | first << 16, T | U << 16)
  int k1 = min((int)sk[lane], kCoderScales - 1);
  int k2 = steps > 1 ? (int)sk[64 + lane] : 0;
  uint2 h1 = shead[k1];
  int16_t* const qs = q + base;
  auto step = [&](int t, auto allc) __attribute__((always_inline)) {
    constexpr bool all = decltype(allc)::value;
    const int li = t * 64 + lane;
    const bool act = all || li < cnt;
    const int row = 257 * k1;
    const int R = (int)(h1.x & 0xFFFFu), o = (int)(h1.x >> 16);
    const uint32_t T = h1.y & 0xFFFFu, U = h1.y >> 16;
    k1 = min(k2, kCoderScales - 1);
    h1 = shead[k1];
    if (t + 2 < steps) k2 = sk[li + 128];
    const uint32_t slot = x & 0xFFFFu;
    // most buckets hold at most one entry boundary, settled by the next start
    const uint16_t* const bk = sbk + row + (slot >> 8);
    int lo = bk[0];
    const int hi = bk[1];
    const uint16_t* const e = sst + o + lo;
    const uint32_t v0 = e[0], v1 = e[1], v2 = e[2];
    const bool up = hi > lo && v1 <= slot;
    uint32_t c = up ? v1 : v0, cn = up ? v2 : v1;
    lo += up ? 1 : 0;
    // slots in the leading or trailing run of frequency-1 entries map to their
    // entry directly; buckets with more boundaries are searched
    const bool run = slot < T || slot >= 65536u - U;
    const bool more = hi > lo && cn <= slot;
    if (__ballot(run || more)) {
      if (more && !run) {
        int h = hi;
        while (lo < h) {
          const int mid = (lo + h + 1) >> 1;
          if (sst[o + mid] <= slot) lo = mid;
          else h = mid - 1;
        }
        c = sst[o + lo];
        cn = sst[o + lo + 1];
      }
      if (run) {
        lo = slot < T ? (int)slot : 2 * R + 2 - 65536 + (int)slot;
        c = slot;
        cn = slot + 1;
      }
    }
    const uint32_t f = (cn - c) & 0xFFFFu;
    const bool esc = act && lo == 2 * R + 1;
    const uint32_t y = __umul24(f, x >> 16) + (slot - c);
    x = act ? y : x;
    refill(act && y < kRansL);
    int qv = lo - R;
    if (__ballot(esc)) {
      const uint32_t fld = x & 0xFFFFu;
      if (esc) x >>= 16;
      refill(esc);
      if (esc) {
        const int mag = R + 1 + (int)(fld & 32767u);
        qv = max(min((fld >> 15) ? -mag : mag, 32767), -32768);
      }
    }
    if (act) qs[li] = (int16_t)qv;
  };
  for (int t = 0; t < steps - 1; ++t) step(t, std::true_type{});
  if (steps > 0) step(steps - 1, std::false_type{});
  if (pos > len) err |= 2;
  if (!bad && (x != kRansL || pos != len)) err |= 4;
  err = wave_or(err);
  uint32_t ticket = 0;
  if (lane == 0) {
    errs[s] = err;
    __threadfence();
    ticket = atomicAdd(count, 1u);
  }
  ticket = (uint32_t)__shfl((int)ticket, 0, 64);
  if (ticket == (uint32_t)ns - 1) {  // every other stream has published its bits
    __threadfence();
    uint32_t all = 0;
    for (int i = lane; i < ns; i += 64) all |= __hip_atomic_load(errs + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    all = wave_or(all);
    if (lane == 0) {
      if (status_out) *status_out = (int32_t)all;
      __hip_atomic_store(count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

hipError_t launch_rans_encode(const RansSections& secs, const uint16_t* tab, uint16_t* scratch, int64_t max_words,
                              uint32_t* lens, hipStream_t st) {
  if (secs.count < 1 || secs.count > kRansMaxSections) return hipErrorInvalidValue;
  int64_t total = 0;
  for (int i = 0; i < secs.count; ++i) {
    if (secs.sec[i].ns <= 0 || secs.sec[i].ns > 65535 || secs.sec[i].ns != rans_streams(secs.sec[i].n)) return hipErrorInvalidValue;
    total += secs.sec[i].ns;
  }
  launch(k_rans_encode, dim3((unsigned)total), dim3(64), st, secs, tab, scratch, max_words, lens);
  launch(k_rans_pack, dim3((unsigned)total), dim3(256), st, secs, (const uint16_t*)scratch, max_words,
         (const uint32_t*)lens);
  return hipGetLastError();
}

hipError_t launch_rans_decode(const uint8_t* in, uint64_t in_bytes, const uint8_t* k, int64_t n, const uint16_t* tab,
                              uint32_t* errs, uint32_t* count, int16_t* q, int32_t* status_out, hipStream_t st) {
  const int64_t ns = (n + kRansStream - 1) / kRansStream;
  if (ns <= 0 || ns > 65535) return hipErrorInvalidValue;
  launch(k_rans_decode, dim3((unsigned)ns), dim3(64), st, in, in_bytes, k, n, tab, errs, count, q, status_out);
  return hipGetLastError();
}

}  // namespace nc
