// Integerised path kernels (Sec. 4.5; Supp. B.4, Alg. 1) for gfx950.
//
// CDNA4 has no int16 matrix instruction, so every int16 x int16 -> int32
// contraction is done exactly on the int8 MFMA: activations split as
// x = 256 xh + xl' + 128 (xh = x >> 8, xl' = (x & 255) - 128) and weights as
// balanced digits w = 256 wh + wl, giving
//   sum x w = 65536 sum xh wh + 256 (sum xh wl + sum xl' wh) + sum xl' wl + 128 sum w.
// Each partial sum fits int32 for K <= 1024; the final combination wraps
// modulo 2^32 exactly like an int32 accumulator, so the result equals the
// exact sum whenever that sum fits int32 (the paper's accumulator contract).
// The 128 sum w term and the bias term 512 b_i are pre-added per output
// channel ("corr").  Every conv then rescales with round-half-to-even of
// a / 8192 and saturates to int16.
#include "common.hpp"
#include "internal.hpp"
#include "pw_load.hpp"

#include <cstring>

namespace nc {

__device__ __forceinline__ uint32_t pack2(int lo, int hi) {
  return ((uint32_t)lo & 0xFFFFu) | ((uint32_t)hi << 16);
}

// The integer sigmoid table S (Sec. 4.5) from its compact form s8, and RHE of
// a / 512 (both described with the gated block below).
constexpr int kSigSat = 888;   // S[v] = 512 from here on
constexpr int kSigBytes = 896; // s8, padded to 16-byte units
__device__ __forceinline__ int dci_sigmoid(int v, const uint8_t* s8) {
  const int a = v < 0 ? -v : v;
  const int sa = a >= kSigSat ? 512 : 256 + (int)s8[min(a, kSigSat - 1)];  // index kept in the table
  return v < 0 ? 512 - sa : sa;
}
// RHE(m / 512) for |m| <= 2^30
__device__ __forceinline__ int rhe9(int m) { return (m + 255 + ((m >> 9) & 1)) >> 9; }

// ---------------------------------------------------------------- pointwise
// Same tiling and LDS pipeline as the fp16 pointwise kernel: 8 waves per tile
// of 128 output pixels, K consumed 64 at a time through three LDS stages.  A
// stage holds the activation slice (int16, or the fp16 frame for the patch
// embed, converted with x_i = round(512 x) when the operand is read) and, per
// 32-row tile, four int8 fragments: hi digits for k-steps 0 and 1, then lo
// digits for k-steps 0 and 1 (32 contraction indices each).
struct PwSmemI {
  static constexpr int ACT = 128 * 128;
};
template <int NT>
struct PwSmemIN {
  static constexpr int WGT = NT / 32 * 4 * 1024;
  static constexpr int STAGE = PwSmemI::ACT + WGT;
  static constexpr int DMA_PER_WAVE = (PwSmemI::ACT / 1024 + WGT / 1024) / 8;
};

template <int NT, int LOADER>
__device__ __forceinline__ void pwi_issue(const PwArgs& a, PwAct<LOADER>& act, int n0, int kc, char* stage, int wave, int lane) {
  act.issue(a, kc, stage, wave);
  const int ks = a.K / 32;
#pragma unroll
  for (int i = 0; i < PwSmemIN<NT>::WGT / 1024 / 8; ++i) {
    const int f = wave + 8 * i;  // row tile f / 4; f % 4: hi k0, hi k1, lo k0, lo k1
    const int mt = n0 / 32 + (f >> 2), sk = 2 * kc + (f & 1);
    const char* plane = (f & 2) ? (const char*)a.wfrag_lo : (const char*)a.wfrag;
    dma16s(plane + ((size_t)mt * ks + sk) * 1024, lane * 16, stage + PwSmemI::ACT + f * 1024);
  }
}

template <int NT, int LOADER>
__device__ __forceinline__ void pwi_compute(const char* stage, int pg, int hf, int lane, intx16 (*acc)[3]) {
  constexpr int RT = NT / 64;
  const int pl = pg * 32 + (lane & 31), h = lane >> 5;
  intx4 bh[2], bl[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    // contraction indices 32 ks + 16 h .. +15 = vectors 4 ks + 2 h and + 1
    const int v0 = 4 * ks + 2 * h;
    uint32_t d[8];
    if constexpr (LOADER == LD_FRAME) {
      const half8 x0 = *(const half8*)(stage + pl * 128 + ((v0 ^ ((pl >> 1) & 7)) << 4));
      const half8 x1 = *(const half8*)(stage + pl * 128 + (((v0 + 1) ^ ((pl >> 1) & 7)) << 4));
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        d[e] = pack2(clip16((int)rintf((float)x0[2 * e] * 512.f)), clip16((int)rintf((float)x0[2 * e + 1] * 512.f)));
        d[4 + e] = pack2(clip16((int)rintf((float)x1[2 * e] * 512.f)), clip16((int)rintf((float)x1[2 * e + 1] * 512.f)));
      }
    } else {
      const intx4 q0 = *(const intx4*)(stage + pl * 128 + ((v0 ^ ((pl >> 1) & 7)) << 4));
      const intx4 q1 = *(const intx4*)(stage + pl * 128 + (((v0 + 1) ^ ((pl >> 1) & 7)) << 4));
#pragma unroll
      for (int e = 0; e < 4; ++e) { d[e] = (uint32_t)q0[e]; d[4 + e] = (uint32_t)q1[e]; }
    }
    split16(d, bh[ks], bl[ks]);
  }
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const char* wt = stage + PwSmemI::ACT + (hf * RT + t) * 4 * 1024 + lane * 16;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const intx4 wh = *(const intx4*)(wt + ks * 1024), wl = *(const intx4*)(wt + (2 + ks) * 1024);
      acc[t][0] = mfma_i8(wh, bh[ks], acc[t][0]);
      acc[t][1] = mfma_i8(wh, bl[ks], acc[t][1]);
      acc[t][1] = mfma_i8(wl, bh[ks], acc[t][1]);
      acc[t][2] = mfma_i8(wl, bl[ks], acc[t][2]);
    }
  }
}

template <int NT, int LOADER, int EPI>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(NT == 64 ? 4 : 2))) void k_pw_i16(PwArgs a) {
  using S = PwSmemIN<NT>;
  constexpr int RT = NT / 64;
  __shared__ __attribute__((aligned(1024))) char st0[S::STAGE];
  __shared__ __attribute__((aligned(1024))) char st1[S::STAGE];
  __shared__ __attribute__((aligned(1024))) char st2[S::STAGE];
  const int ntile = (a.P + 127) / 128;
  // (tile, row pass) pairs with the row pass fastest, each XCD taking a
  // contiguous range: the passes over one pixel tile run together and share
  // its activations in L2.
  const int npass = a.N / NT;
  const int lin = xcd_tile(blockIdx.x, gridDim.x);
  const int tile = lin / npass;
  if (tile >= ntile) return;
  // the upsample that follows the prior in an encode: workgroup 0 first adds
  // up the frame's rate partials
  if constexpr (EPI == EP_UP)
    if (a.bits_out && blockIdx.x == 0) block_sum_to(a.sum_base, a.n_sum, a.bits_out);
  const int lane = threadIdx.x & 63, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int pg = wave & 3, hf = wave >> 2;
  const int n0 = (lin - tile * npass) * NT;
  const int nk = a.K / 64;

  intx16 acc[RT][3];
#pragma unroll
  for (int t = 0; t < RT; ++t) acc[t][0] = acc[t][1] = acc[t][2] = intx16{};
  intx4 corr[RT][4];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int g = 0; g < 4; ++g) corr[t][g] = *(const intx4*)((const int*)a.bias + n0 + 32 * (hf * RT + t) + 8 * g + 4 * h);

  PwAct<LOADER> act;
  act.init(a, tile, n0, wave, lane);
  pwi_issue<NT, LOADER>(a, act, n0, 0, st0, wave, lane);
  if (nk > 1) pwi_issue<NT, LOADER>(a, act, n0, 1, st1, wave, lane);
  auto step = [&](int kc, const char* cur, char* refill) {
    const int ahead = min(nk - 1 - kc, 1);  // stages issued after kc still in flight
    if (ahead == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(S::DMA_PER_WAVE) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();
    if (kc + 2 < nk) pwi_issue<NT, LOADER>(a, act, n0, kc + 2, refill, wave, lane);
    pwi_compute<NT, LOADER>(cur, pg, hf, lane, acc);
  };
  for (int kc = 0; kc < nk; kc += 3) {
    step(kc, st0, st2);
    if (kc + 1 < nk) step(kc + 1, st1, st0);
    if (kc + 2 < nk) step(kc + 2, st2, st1);
  }
  lds_barrier();

  // park the rescaled int16 results as int32, as in the fp16 kernel
  constexpr int SWZ = (NT / 4 - 1) & 31;
  // pixel group g parks at offset (g % GPS) * PARK of stage g / GPS
  constexpr int PARK = 32 * NT * 4, GPS = S::STAGE / PARK;
  static_assert(GPS >= 2, "four pixel groups fit three stage buffers");
  auto park = [&](int g) __attribute__((always_inline)) -> char* {
    return (g / GPS == 0 ? st0 : g / GPS == 1 ? st1 : st2) + (g % GPS) * PARK;
  };
  {
    char* ob = park(pg);
    const int row = lane & 31;
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int nl = 32 * (hf * RT + t) + 8 * g + 4 * h;
        intx4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int r = 4 * g + e;
          o[e] = rescale13(combine_i16(acc[t][0][r], acc[t][1][r], acc[t][2][r], corr[t][g][e]));
        }
        *(intx4*)(ob + row * (NT * 4) + (((nl >> 2) ^ (row & SWZ)) << 4)) = o;
      }
  }
  // prior head: a pass covers channels c0 .. c0+31 (rows 0-31 mu_i, 32-63 s_i);
  // the tile's symbols are staged in stage buffer 2 as [channel][pixel]
  const int c0 = a.c_off + n0 / 2;
  int16_t* qt = (int16_t*)st2;
  uint8_t* kt = (uint8_t*)(st2 + 8192);  // scale indices, [channel][pixel]
  // planar store of the staged scale indices (after a barrier)
  auto store_k = [&]() __attribute__((always_inline)) {
    const int ch = threadIdx.x >> 4, k = threadIdx.x & 15;
    const int p0 = tile * 128 + 8 * k;
    uint8_t* dk = a.k_out + (size_t)(c0 + ch) * a.P + p0;
    const uint8_t* sk = kt + ch * 128 + 8 * k;
    if ((a.P & 7) == 0 && p0 + 8 <= a.P && ((uintptr_t)a.k_out & 7) == 0) {
      *(uint64_t*)dk = *(const uint64_t*)sk;
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (p0 + e < a.P) dk[e] = sk[e];
    }
  };
  if constexpr (EPI == EP_PRIOR_DEC) {
    static_assert(NT == 64, "prior passes are 64 rows");
    const int ch = threadIdx.x >> 4, k = threadIdx.x & 15;
    const int p0 = tile * 128 + 8 * k;
    const int16_t* src = a.q_in + (size_t)(c0 + ch) * a.P + p0;
    shortx8 v = {};
    if ((a.P & 7) == 0 && p0 + 8 <= a.P) {
      v = *(const shortx8*)src;
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = p0 + e < a.P ? src[e] : (short)0;
    }
    *(shortx8*)(qt + ch * 128 + 8 * k) = v;
  }
  lds_barrier();

  auto parked = [&](int px, int nl8, int* v) {
    const int gpx = px >> 5, row = px & 31;
    const char* ob = park(gpx);
    const intx4 o0 = *(const intx4*)(ob + row * (NT * 4) + (((2 * nl8) ^ (row & SWZ)) << 4));
    const intx4 o1 = *(const intx4*)(ob + row * (NT * 4) + (((2 * nl8 + 1) ^ (row & SWZ)) << 4));
#pragma unroll
    for (int e = 0; e < 4; ++e) { v[e] = o0[e]; v[4 + e] = o1[e]; }
  };
  constexpr int UNITS = 128 * (NT / 8);
  // (mu_i, s_i) of 8 channels c .. c + 7 of pixel gp: the head's rows plus,
  // saturating, the addend of the two-step entropy model (hyper parameters,
  // or the first step's (mu_i, s_i) for the second step)
  auto prior_ms = [&](int px, int g8, int gp, int* mu, int* sv) __attribute__((always_inline)) {
    parked(px, g8, mu);
    parked(px, 4 + g8, sv);
    if (a.add && gp < a.P) {
      const size_t at = (size_t)gp * a.add_ld + (c0 + 8 * g8 - a.add_c0);
      const shortx8 hm = *(const shortx8*)((const int16_t*)a.add + at);
      const shortx8 hs = *(const shortx8*)((const int16_t*)a.add + at + a.add_s);
#pragma unroll
      for (int e = 0; e < 8; ++e) { mu[e] = clip16(mu[e] + (int)hm[e]); sv[e] = clip16(sv[e] + (int)hs[e]); }
    }
  };
  // channels >= split: (mu_i, s_i) go to the base buffer for the second step
  const bool to_base = a.split && c0 >= a.split;
  auto store_base = [&](int g8, int gp, const int* mu, const int* sv) __attribute__((always_inline)) {
    if (gp >= a.P) return;
    const int nb = a.Cdst - a.split;
    int16_t* b = (int16_t*)a.base + (size_t)gp * 2 * nb + (c0 + 8 * g8 - a.split);
    shortx8 m, v;
#pragma unroll
    for (int e = 0; e < 8; ++e) { m[e] = (short)mu[e]; v[e] = (short)sv[e]; }
    *(shortx8*)b = m;
    *(shortx8*)(b + nb) = v;
  };
  if constexpr (EPI == EP_SCALES) {
    const int px = threadIdx.x >> 2, g8 = threadIdx.x & 3;
    const int gp = tile * 128 + px;
    int mu[8], sv[8];
    prior_ms(px, g8, gp, mu, sv);
    if (to_base) {
      store_base(g8, gp, mu, sv);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) kt[(8 * g8 + e) * 128 + px] = a.k_tab[sv[e] + 32768];
      // mu_i (int16, NHWC), for yhat_i = clip(512 q + mu_i) once the symbols are decoded
      if (a.dst && gp < a.P) {
        shortx8 m;
#pragma unroll
        for (int e = 0; e < 8; ++e) m[e] = (short)mu[e];
        *(shortx8*)((int16_t*)a.dst + (size_t)gp * a.Cdst + c0 + 8 * g8) = m;
      }
    }
    lds_barrier();
    if (!to_base) store_k();
  } else if constexpr (EPI == EP_PRIOR || EPI == EP_PRIOR_DEC) {
    // thread = (pixel px, 8 channels g8): q = RHE((y_i - mu_i) / 512),
    // yhat_i = clip(512 q + mu_i), sigma from the table at s_i
    const int px = threadIdx.x >> 2, g8 = threadIdx.x & 3;
    const int gp = tile * 128 + px;
    const int c = c0 + 8 * g8;
    int mu[8], sv[8];
    prior_ms(px, g8, gp, mu, sv);
    if (to_base) {
      store_base(g8, gp, mu, sv);
      if constexpr (EPI == EP_PRIOR)
        if (threadIdx.x == 0) a.partials[(size_t)tile * npass + n0 / NT] = 0.0;
    } else if constexpr (EPI == EP_PRIOR) {
      double bsum = 0.0;
      shortx8 yv = {};
      if (gp < a.P) yv = *(const shortx8*)((const int16_t*)a.y + (size_t)gp * a.Cdst + c);
      shortx8 yh;
      if (a.k_out) {
#pragma unroll
        for (int e = 0; e < 8; ++e) kt[(8 * g8 + e) * 128 + px] = a.k_tab[sv[e] + 32768];
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int q = rhe_shift((int)yv[e] - mu[e], 9);
        qt[(8 * g8 + e) * 128 + px] = (int16_t)q;
        yh[e] = (short)clip16(512 * q + mu[e]);
        if (gp < a.P) bsum += (double)symbol_bits((float)q, a.sigma_tab[sv[e] + 32768]);
      }
      if (gp < a.P) *(shortx8*)((int16_t*)a.dst + (size_t)gp * a.Cdst + c) = yh;
      __shared__ double red[8];
      bsum = wave_sum(bsum);
      if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = bsum;
      lds_barrier();
      {
        const int ch = threadIdx.x >> 4, k = threadIdx.x & 15;
        const int p0 = tile * 128 + 8 * k;
        const shortx8 v = *(const shortx8*)(qt + ch * 128 + 8 * k);
        int16_t* dq = a.q_out + (size_t)(c0 + ch) * a.P + p0;
        if ((a.P & 7) == 0 && p0 + 8 <= a.P) {
          *(shortx8*)dq = v;
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (p0 + e < a.P) dq[e] = v[e];
        }
      }
      if (a.k_out) store_k();
      if (threadIdx.x == 0) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < 8; ++w) t += red[w];
        a.partials[(size_t)tile * npass + n0 / NT] = t;
      }
    } else {
      if (gp < a.P) {
        shortx8 yh;
#pragma unroll
        for (int e = 0; e < 8; ++e) yh[e] = (short)clip16(512 * (int)qt[(8 * g8 + e) * 128 + px] + mu[e]);
        *(shortx8*)((int16_t*)a.dst + (size_t)gp * a.Cdst + c) = yh;
      }
    }
  } else if constexpr (EPI == EP_ZQUANT) {
    // the 64 rows are the channels of z_i: q_z = RHE(z_i / 512) (staged
    // [channel][pixel] in stage buffer 2, 16 KiB), zhat_i = clip(512 q_z)
    // (NHWC), rate under sigma_z[c]
    static_assert(NT == 64, "z has 64 channels");
    const int px = threadIdx.x >> 2, g8 = threadIdx.x & 3;
    const int gp = tile * 128 + px;
    double bsum = 0.0;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int cz = 32 * half + 8 * g8;
      int zv[8];
      parked(px, 4 * half + g8, zv);
      shortx8 zh;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int q = rhe_shift(zv[e], 9);
        qt[(cz + e) * 128 + px] = (int16_t)q;
        zh[e] = (short)clip16(512 * q);
        if (gp < a.P) bsum += (double)symbol_bits((float)q, a.zsigma[cz + e]);
      }
      if (gp < a.P) *(shortx8*)((int16_t*)a.dst + (size_t)gp * a.Cdst + cz) = zh;
    }
    __shared__ double redz[8];
    bsum = wave_sum(bsum);
    if ((threadIdx.x & 63) == 0) redz[threadIdx.x >> 6] = bsum;
    lds_barrier();
#pragma unroll
    for (int it = 0; it < 2; ++it) {
      const int ch = 32 * it + (threadIdx.x >> 4), k = threadIdx.x & 15;
      const int p0 = tile * 128 + 8 * k;
      const shortx8 v = *(const shortx8*)(qt + ch * 128 + 8 * k);
      int16_t* dq = a.q_out + (size_t)ch * a.P + p0;
      if ((a.P & 7) == 0 && p0 + 8 <= a.P) {
        *(shortx8*)dq = v;
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (p0 + e < a.P) dq[e] = v[e];
      }
    }
    if (threadIdx.x == 0) {
      double t = 0.0;
#pragma unroll
      for (int w = 0; w < 8; ++w) t += redz[w];
      a.partials[tile] = t;
    }
  } else if constexpr (EPI == EP_GATE) {
    // rows 64 j .. + 31 of the pass: h1 of gated channels n0 / 2 + 32 j .. + 31,
    // rows 64 j + 32 .. + 63: the matching h2.  As the fused gated block:
    // WSiLU_i = RHE(h1 S[h1] / 512), g = clip(RHE(WSiLU_i h2 / 512)).
    constexpr int G = NT / 64, GU = 128 * G * 4;  // units (pixel, group, 8 channels)
#pragma unroll
    for (int it = 0; it < GU / 512; ++it) {
      const int idx = it * 512 + threadIdx.x;
      const int px = idx / (4 * G), j = (idx >> 2) % G, g8 = idx & 3;
      const int gp = tile * 128 + px;
      if (gp < a.P) {
        int h1[8], h2[8];
        parked(px, 8 * j + g8, h1);
        parked(px, 8 * j + 4 + g8, h2);
        shortx8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int w1 = rhe9(h1[e] * dci_sigmoid(h1[e], a.sig8));  // |h S| <= 2^24
          o[e] = (short)clip16(rhe9(w1 * h2[e]));                    // |product| <= 2^30
        }
        *(shortx8*)((int16_t*)a.dst + (size_t)gp * a.Cdst + n0 / 2 + 32 * j + 8 * g8) = o;
      }
    }
  } else if constexpr (EPI == EP_REC) {
#pragma unroll
    for (int it = 0; it < UNITS / 512; ++it) {
      const int idx = it * 512 + threadIdx.x;
      const int nl8 = idx >> 7, px = idx & 127;
      const int gp = tile * 128 + px;
      if (gp < a.P) {
        int v[8];
        parked(px, nl8, v);
        const int n = n0 + 8 * nl8, c = n >> 6, i = (n >> 3) & 7;
        const int py = gp / a.w8, pxx = gp - py * a.w8;
        shortx8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (short)min(max(v[e], 0), 512);
        *(shortx8*)((int16_t*)a.dst + (size_t)c * a.H * a.W + (size_t)(8 * py + i) * a.W + 8 * pxx) = o;
      }
    }
  } else {
#pragma unroll
    for (int it = 0; it < UNITS / 512; ++it) {
      const int idx = it * 512 + threadIdx.x;
      const int px = idx / (NT / 8), nl8 = idx % (NT / 8);
      const int gp = tile * 128 + px;
      if (gp < a.P) {
        int v[8];
        parked(px, nl8, v);
        shortx8 o;
        if constexpr (EPI == EP_LRELU) {
          // integer LeakyReLU, slope RHE(0.1 * 2^13) = 819: max(h, RHE(819 h / 2^13))
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int m = 819 * v[e];
            o[e] = (short)max(v[e], (m + 4095 + ((m >> 13) & 1)) >> 13);
          }
        } else if constexpr (EPI == EP_RESID) {
          // saturating residual add
          const shortx8 zr = *(const shortx8*)((const int16_t*)a.res + (size_t)gp * a.Cdst + n0 + 8 * nl8);
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = (short)clip16((int)zr[e] + v[e]);
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = (short)v[e];
        }
        size_t off;
        if constexpr (EPI == EP_NHWC || EPI == EP_LRELU || EPI == EP_RESID) {
          off = (size_t)gp * a.Cdst + n0 + 8 * nl8;
        } else {
          const int C = a.Cdst, n = n0 + 8 * nl8;
          const int sp = n / C, c = n - sp * C;
          const int w16 = a.w8 >> 1;
          const int Y = gp / w16, X = gp - Y * w16;
          off = (size_t)((2 * Y + (sp >> 1)) * a.w8 + 2 * X + (sp & 1)) * C + c;
        }
        *(shortx8*)((int16_t*)a.dst + off) = o;
      }
    }
  }
}

template <int NT>
static hipError_t pw_dispatch(int loader, int epi, const PwArgs& a, hipStream_t st) {
  dim3 grid(grid_tiles(a.P) * (a.N / NT)), block(512);
#define NC_PW(L, E)                                                            \
  if (loader == L && epi == E) {                                               \
    launch(k_pw_i16<NT, L, E>, grid, block, st, a);                            \
    return hipGetLastError();                                                  \
  }
  NC_PW(LD_NHWC, EP_NHWC)
  NC_PW(LD_FRAME, EP_NHWC)
  NC_PW(LD_DOWN, EP_NHWC)
  NC_PW(LD_NHWC, EP_UP)
  NC_PW(LD_NHWC, EP_REC)
  NC_PW(LD_NHWC, EP_LRELU)
  NC_PW(LD_NHWC, EP_RESID)
  NC_PW(LD_NHWC, EP_GATE)
  if constexpr (NT == 64) {  // epilogues that pair two 32-row halves of a pass
    NC_PW(LD_NHWC, EP_PRIOR)
    NC_PW(LD_NHWC, EP_PRIOR_DEC)
    NC_PW(LD_NHWC, EP_SCALES)
    NC_PW(LD_DOWN, EP_ZQUANT)
  }
#undef NC_PW
  return hipErrorInvalidValue;
}

// 64 rows per workgroup pass: two workgroups fit a CU, and the passes over one
// pixel tile run side by side on one XCD.  K must be a multiple of 64 (C = 64,
// 128, 256; 192 for the patch embed) and N a multiple of 64.
hipError_t launch_pw_i16(int loader, int epi, const PwArgs& a, hipStream_t st) {
  if (a.K % 64 || a.N % 64) return hipErrorInvalidValue;
  // 128 rows per pass for the patch embed and the 2C -> C fuse: their activation
  // tiles are the widest (K = 192 frame values or 2C channels), so halving the
  // passes that re-stage them pays, and they still have two passes per tile.
  if (a.N % 128 == 0 && epi == EP_NHWC && (loader == LD_FRAME || (loader == LD_NHWC && a.K >= 512)))
    return pw_dispatch<128>(loader, epi, a, st);
  // the two halves of a wide DC block (C > 256) at 1/8 scale: 128-row passes
  if ((epi == EP_LRELU || epi == EP_RESID || epi == EP_GATE) && a.N % 128 == 0)
    return pw_dispatch<128>(loader, epi, a, st);
  return pw_dispatch<64>(loader, epi, a, st);
}

// Integer prior head, quantiser q = RHE((y_i - mu_i) / 512),
// yhat_i = clip(512 q + mu_i) and bits with sigma looked up from the
// 65536-entry table indexed by s_i (Supp. B.2, Alg. 1), as the epilogue of the
// pointwise kernel over passes of 32 mu rows + the 32 s rows of the same
// channels.  Bit partial sums: one per (tile, pass).
int prior_partials_i16(int C, int P) { return ((P + 127) / 128) * (C / 32); }

hipError_t launch_prior_i16(const PriorArgs& pa, hipStream_t st, int* n_partials) {
  if (pa.C % 32) return hipErrorInvalidValue;
  PwArgs a;
  std::memset(&a, 0, sizeof(a));
  a.wfrag = pa.wfrag;
  a.wfrag_lo = pa.wfrag_lo;
  a.bias = pa.bias;
  a.K = pa.K ? pa.K : pa.C;
  a.N = pa.N ? pa.N : 2 * pa.C;
  a.ld0 = pa.ld0;
  a.c_off = pa.c_off;
  a.add = pa.add;
  a.add_ld = pa.add_ld;
  a.add_s = pa.add_s;
  a.add_c0 = pa.add_c0;
  a.split = pa.split;
  a.base = pa.base;
  a.P = pa.P;
  a.src0 = pa.yhat_prev;
  a.C0 = a.K;
  a.dst = pa.decode == 2 ? pa.mu_out : pa.yhat_new;
  a.Cdst = pa.C;
  a.y = pa.y;
  a.q_in = pa.q_in;
  a.q_out = pa.q_out;
  a.partials = pa.partials;
  a.sigma_tab = pa.sigma_tab;
  a.k_out = pa.k_out;
  a.k_tab = pa.k_tab;
  if (n_partials) *n_partials = ((pa.P + 127) / 128) * (a.N / 64);
  return pw_dispatch<64>(LD_NHWC, pa.decode == 2 ? EP_SCALES : pa.decode ? EP_PRIOR_DEC : EP_PRIOR, a, st);
}

hipError_t launch_zquant_i16(const PwArgs& a, hipStream_t st, int* n_partials) {
  if (a.N != 64 || a.K % 64) return hipErrorInvalidValue;
  if (n_partials) *n_partials = (a.P + 127) / 128;
  return pw_dispatch<64>(LD_DOWN, EP_ZQUANT, a, st);
}

}  // namespace nc
