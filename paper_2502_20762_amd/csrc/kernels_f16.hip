// fp16 path kernels (fp16 storage, fp32 MFMA accumulation) for gfx950.
//
// k_pw_f16      pointwise / patch-embed / 2x2-s2 / upsample / reconstruction
//               contractions (out^T = W * act^T + b) with gather-on-load and
//               scatter-on-store, and the prior head with the quantiser and
//               the bit partial sums as its epilogue (Fig. 4 "Q", Supp. B.2).
// The larger contractions are in kernels_f16_pwt.hip, the DC blocks in
// kernels_f16_dc64.hip and kernels_f16_dc128.hip.
#include "common.hpp"
#include "internal.hpp"
#include "pw_load.hpp"

#include <cstring>
#include <type_traits>
#include <utility>

namespace nc {

// f(integral_constant<int, T>) for every T of the sequence, in order
template <typename F, int... T>
__device__ __forceinline__ void unrolled_steps(F& f, std::integer_sequence<int, T...>) {
  (f(std::integral_constant<int, T>{}), ...);
}

// ---------------------------------------------------------------- pointwise
// out^T[rows n0 .. n0+NT)[128 pixels] = W * act^T (+ bias) for one tile of
// 128 consecutive output pixels.  8 waves: wave w owns pixels 32 (w & 3) ..
// +31 and rows (w >> 2) NT/2 .. +NT/2.  K is consumed 64 at a time through three
// LDS stages (distinct objects, statically indexed), each holding the
// activation slice (128 pixels x 64 channels, one 128-byte row per pixel,
// 16-byte vector v of pixel px stored at slot v ^ ((px / 2) & 7), which keeps
// the 16 lanes of each quarter of a B-fragment read on distinct banks) and the weight
// fragments of those 64 contraction indices, filled by direct global->LDS
// loads two stages ahead.  Three stages leave room for two workgroups per CU,
// so one workgroup's load latency and stores overlap the other's MFMA work.
// The result is parked in LDS and written with coalesced 16-byte stores.
template <int NT>
struct PwSmem {
  static constexpr int ACT = 128 * 128;               // activation slice bytes
  static constexpr int WGT = NT / 32 * 4 * 1024;      // weight fragments bytes
  static constexpr int STAGE = ACT + WGT;
  static constexpr int DMA_PER_WAVE = (ACT / 1024 + WGT / 1024) / 8;
};

template <int NT, int LOADER>
__device__ __forceinline__ void pw_issue(const PwArgs& a, PwAct<LOADER>& act, int n0, int kc, char* stage, int wave, int lane) {
  using S = PwSmem<NT>;
  act.issue(a, kc, stage, wave);
  const int ks = a.K / 16;
#pragma unroll
  for (int i = 0; i < S::WGT / 1024 / 8; ++i) {
    const int f = wave + 8 * i;  // fragment f of the stage: row tile f / 4, k-step f % 4
    const int mt = n0 / 32 + (f >> 2), sk = 4 * kc + (f & 3);
    dma16s((const char*)a.wfrag + ((size_t)mt * ks + sk) * 1024, lane * 16, stage + S::ACT + f * 1024);
  }
}

template <int NT>
__device__ __forceinline__ void pw_compute(const char* stage, int pg, int hf, int lane, floatx16* acc) {
  using S = PwSmem<NT>;
  constexpr int RT = NT / 64;  // row tiles per wave
  const int pl = pg * 32 + (lane & 31), h = lane >> 5;
  half8 b[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) b[ks] = *(const half8*)(stage + pl * 128 + ((((2 * ks + h) ^ ((pl >> 1) & 7))) << 4));
  half8 w[RT][4];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) w[t][ks] = *(const half8*)(stage + S::ACT + ((hf * RT + t) * 4 + ks) * 1024 + lane * 16);
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
#pragma unroll
    for (int t = 0; t < RT; ++t) acc[t] = mfma_f16(w[t][ks], b[ks], acc[t]);
}

template <int NT, int LOADER, int EPI>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(NT == 64 ? 4 : 2))) void k_pw_f16(PwArgs a) {
  using S = PwSmem<NT>;
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

  floatx16 acc[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) acc[t] = floatx16{};
  floatx4 bias[RT][4];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int g = 0; g < 4; ++g) bias[t][g] = *(const floatx4*)((const float*)a.bias + n0 + 32 * (hf * RT + t) + 8 * g + 4 * h);

  PwAct<LOADER> act;
  act.init(a, tile, n0, wave, lane);
  pw_issue<NT, LOADER>(a, act, n0, 0, st0, wave, lane);
  if (nk > 1) pw_issue<NT, LOADER>(a, act, n0, 1, st1, wave, lane);
  // Stage kc: wait until at most the later-issued stages are in flight, make
  // every wave's loads visible, refill the buffer freed in the previous
  // iteration with stage kc + 3, then compute.
  auto step = [&](int kc, const char* cur, char* refill) {
    const int ahead = min(nk - 1 - kc, 1);  // stages issued after kc still in flight
    if (ahead == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(S::DMA_PER_WAVE) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();
    if (kc + 2 < nk) pw_issue<NT, LOADER>(a, act, n0, kc + 2, refill, wave, lane);
    pw_compute<NT>(cur, pg, hf, lane, acc);
  };
  for (int kc = 0; kc < nk; kc += 3) {
    step(kc, st0, st2);
    if (kc + 1 < nk) step(kc + 1, st1, st0);
    if (kc + 2 < nk) step(kc + 2, st2, st1);
  }
  lds_barrier();  // every wave is done reading the stages

  // park acc + bias as fp32, one row of NT floats per tile pixel, 16-byte
  // chunk c of the row of pixel px at c ^ (px & SWZ); the 128 rows fill the
  // stage buffers in order, RPB rows per buffer
  constexpr int SWZ = (NT / 4 - 1) & 31;
  constexpr int ROW = NT * 4, RPB = S::STAGE / ROW;
  static_assert(3 * RPB >= 128, "the tile's rows fit three stage buffers");
  auto park_row = [&](int px) __attribute__((always_inline)) -> char* {
    const int b = px / RPB, r = px - b * RPB;
    return (b == 0 ? st0 : b == 1 ? st1 : st2) + r * ROW;
  };
  {
    const int row = lane & 31;
    char* ob = park_row(32 * pg + row);
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int nl = 32 * (hf * RT + t) + 8 * g + 4 * h;  // row of the pass
        floatx4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = acc[t][4 * g + e] + bias[t][g][e];
        *(floatx4*)(ob + (((nl >> 2) ^ (row & SWZ)) << 4)) = o;
      }
  }
  // prior head: a pass covers channels c0 .. c0+31 (rows 0-31 mu, 32-63 s);
  // the tile's symbols are staged in stage buffer 2 as [channel][pixel]
  const int c0 = a.c_off + n0 / 2;
  int16_t* qt = (int16_t*)st2;
  uint8_t* kt = (uint8_t*)(st2 + 8192);  // scale indices, [channel][pixel]
  float* sct = (float*)(st2 + 12288);    // the coder scales, for the scale-index search
  if constexpr (EPI == EP_SCALES || EPI == EP_PRIOR) {
    if (threadIdx.x < kCoderScales && a.k_out) sct[threadIdx.x] = a.scales[threadIdx.x];
  }
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
    const int ch = threadIdx.x >> 4, k = threadIdx.x & 15;  // 32 channels x 16 chunks of 8 pixels
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

  auto parked = [&](int px, int nl8) {  // 8 floats: pass rows nl8 * 8 .. +7 of tile pixel px
    const int row = px & 31;
    const char* ob = park_row(px);
    const floatx4 o0 = *(const floatx4*)(ob + (((2 * nl8) ^ (row & SWZ)) << 4));
    const floatx4 o1 = *(const floatx4*)(ob + (((2 * nl8 + 1) ^ (row & SWZ)) << 4));
    floatx16 r;  // only [0, 8) used
#pragma unroll
    for (int e = 0; e < 4; ++e) { r[e] = o0[e]; r[4 + e] = o1[e]; }
    return r;
  };
  // (mu, s) of 8 channels c .. c + 7 of pixel gp: the head's rows plus the
  // addend of the two-step entropy model (hyper parameters, or the first
  // step's (mu, s) for the second step)
  auto prior_ms = [&](int px, int g8, int gp, float* mu, float* sg) __attribute__((always_inline)) {
    const floatx16 m = parked(px, g8), sv = parked(px, 4 + g8);
#pragma unroll
    for (int e = 0; e < 8; ++e) { mu[e] = m[e]; sg[e] = sv[e]; }
    if (a.add && gp < a.P) {
      const size_t at = (size_t)gp * a.add_ld + (c0 + 8 * g8 - a.add_c0);
      if (a.add_f32) {
        const float* am = (const float*)a.add + at;
#pragma unroll
        for (int e = 0; e < 8; ++e) { mu[e] += am[e]; sg[e] += am[a.add_s + e]; }
      } else {
        const half8 hm = *(const half8*)((const f16*)a.add + at), hs = *(const half8*)((const f16*)a.add + at + a.add_s);
#pragma unroll
        for (int e = 0; e < 8; ++e) { mu[e] += (float)hm[e]; sg[e] += (float)hs[e]; }
      }
    }
  };
  // channels >= split: (mu, s) go to the base buffer for the second step
  const bool to_base = a.split && c0 >= a.split;
  auto store_base = [&](int g8, int gp, const float* mu, const float* sg) __attribute__((always_inline)) {
    if (gp >= a.P) return;
    const int nb = a.Cdst - a.split;
    float* b = (float*)a.base + (size_t)gp * 2 * nb + (c0 + 8 * g8 - a.split);
    *(floatx4*)b = floatx4{mu[0], mu[1], mu[2], mu[3]};
    *(floatx4*)(b + 4) = floatx4{mu[4], mu[5], mu[6], mu[7]};
    *(floatx4*)(b + nb) = floatx4{sg[0], sg[1], sg[2], sg[3]};
    *(floatx4*)(b + nb + 4) = floatx4{sg[4], sg[5], sg[6], sg[7]};
  };
  if constexpr (EPI == EP_SCALES) {
    const int px = threadIdx.x >> 2, g8 = threadIdx.x & 3;
    const int gp = tile * 128 + px;
    float mu[8], sg[8];
    prior_ms(px, g8, gp, mu, sg);
    if (to_base) {
      store_base(g8, gp, mu, sg);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) kt[(8 * g8 + e) * 128 + px] = (uint8_t)coder_scale_index(softplus_sigma(sg[e]), sct);
      // mu as fp32 (NHWC), for yhat = q + mu once the symbols are decoded
      if (a.dst && gp < a.P) {
        float* dm = (float*)a.dst + (size_t)gp * a.Cdst + c0 + 8 * g8;
        *(floatx4*)dm = floatx4{mu[0], mu[1], mu[2], mu[3]};
        *(floatx4*)(dm + 4) = floatx4{mu[4], mu[5], mu[6], mu[7]};
      }
    }
    lds_barrier();
    if (!to_base) store_k();
  } else if constexpr (EPI == EP_PRIOR || EPI == EP_PRIOR_DEC) {
    // thread = (pixel px, 8 channels g8): mu and s from the park, y / q, yhat
    const int px = threadIdx.x >> 2, g8 = threadIdx.x & 3;
    const int gp = tile * 128 + px;
    const int c = c0 + 8 * g8;
    float mu[8], sg[8];
    prior_ms(px, g8, gp, mu, sg);
    double bsum = 0.0;
    if (to_base) {
      store_base(g8, gp, mu, sg);
      if constexpr (EPI == EP_PRIOR)
        if (threadIdx.x == 0) a.partials[(size_t)tile * npass + n0 / NT] = 0.0;
    } else if constexpr (EPI == EP_PRIOR) {
      if (a.k_out) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          kt[(8 * g8 + e) * 128 + px] = (uint8_t)coder_scale_index(softplus_sigma(sg[e]), sct);
      }
      half8 yv = {};
      if (gp < a.P) yv = *(const half8*)((const f16*)a.y + (size_t)gp * a.Cdst + c);
      half8 yh;
      float b8 = 0.f;  // the thread's 8 symbols in fp32, then the fixed-order double sums
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float q = rintf((float)yv[e] - mu[e]);
        q = fminf(fmaxf(q, -32768.f), 32767.f);
        qt[(8 * g8 + e) * 128 + px] = (int16_t)q;
        yh[e] = (f16)(q + mu[e]);
        b8 += symbol_bits(q, softplus_sigma(sg[e]));
      }
      if (gp < a.P) bsum = (double)b8;
      if (gp < a.P) *(half8*)((f16*)a.dst + (size_t)gp * a.Cdst + c) = yh;
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
        half8 yh;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          // same operation order as the encoder: mu first, then q + mu
          const float q = (float)qt[(8 * g8 + e) * 128 + px];
          yh[e] = (f16)(q + mu[e]);
        }
        *(half8*)((f16*)a.dst + (size_t)gp * a.Cdst + c) = yh;
      }
    }
  } else if constexpr (EPI == EP_ZQUANT) {
    // the 64 rows are the channels of z: q_z = round(z) (staged [channel][pixel]
    // in stage buffer 2, 16 KiB), zhat = q_z (NHWC), rate under sigma_z[c]
    static_assert(NT == 64, "z has 64 channels");
    const int px = threadIdx.x >> 2, g8 = threadIdx.x & 3;
    const int gp = tile * 128 + px;
    double bsum = 0.0;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int cz = 32 * half + 8 * g8;
      const floatx16 zv = parked(px, 4 * half + g8);
      half8 zh;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float q = rintf(zv[e]);
        q = fminf(fmaxf(q, -32768.f), 32767.f);
        qt[(cz + e) * 128 + px] = (int16_t)q;
        zh[e] = (f16)q;
        if (gp < a.P) bsum += (double)symbol_bits(q, a.zsigma[cz + e]);
      }
      if (gp < a.P) *(half8*)((f16*)a.dst + (size_t)gp * a.Cdst + cz) = zh;
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
  } else {
    constexpr int UNITS = 128 * (NT / 8);
#pragma unroll
    for (int it = 0; it < UNITS / 512; ++it) {
      const int idx = it * 512 + threadIdx.x;
      const int px = idx / (NT / 8), nl8 = idx % (NT / 8);  // consecutive threads walk a pixel's row
      const int gp = tile * 128 + px;
      if (gp < a.P) {
        const floatx16 r = parked(px, nl8);
        half8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (f16)r[e];
        size_t off;
        if constexpr (EPI == EP_NHWC) {
          off = (size_t)gp * a.Cdst + n0 + 8 * nl8;
        } else {  // EP_UP: pass rows n = sp * C + c, all in one sub-position sp
          const int C = a.Cdst, n = n0 + 8 * nl8;
          const int sp = n / C, c = n - sp * C;
          const int w16 = a.w8 >> 1;
          const int Y = gp / w16, X = gp - Y * w16;
          off = (size_t)((2 * Y + (sp >> 1)) * a.w8 + 2 * X + (sp & 1)) * C + c;
        }
        *(half8*)((f16*)a.dst + off) = o;
      }
    }
  }
}

template <int NT>
static hipError_t pw_dispatch(int loader, int epi, const PwArgs& a, hipStream_t st) {
  dim3 grid(grid_tiles(a.P) * (a.N / NT)), block(512);
#define NC_PW(L, E)                                                            \
  if (loader == L && epi == E) {                                               \
    launch(k_pw_f16<NT, L, E>, grid, block, st, a);                            \
    return hipGetLastError();                                                  \
  }
  NC_PW(LD_FRAME_CTX, EP_NHWC)
  NC_PW(LD_DOWN, EP_NHWC)
  NC_PW(LD_NHWC, EP_UP)
  NC_PW(LD_UP_CTX, EP_UP)
  NC_PW(LD_NHWC, EP_PRIOR)
  NC_PW(LD_NHWC, EP_PRIOR_DEC)
  NC_PW(LD_NHWC, EP_SCALES)
  NC_PW(LD_DOWN, EP_ZQUANT)
#undef NC_PW
  return hipErrorInvalidValue;
}

// 64 rows per workgroup pass: two workgroups fit a CU, and the passes over one
// pixel tile run side by side on one XCD.  K must be a multiple of 64 (C = 64,
// 128, 256; 192 for the patch embed) and N a multiple of 64.
hipError_t launch_pw_f16(int loader, int epi, const PwArgs& a, hipStream_t st) {
  if (a.K % 64 || a.N % 64) return hipErrorInvalidValue;
  // the reconstruction, from C = 128 on the folded input convs and above C = 256 the
  // two halves of a DC block: large register tiles
  if (((loader == LD_FRAME_CTX || loader == LD_UP_CTX) && a.Cdst % 128 == 0) || epi == EP_REC || epi == EP_LRELU ||
      epi == EP_RESID || epi == EP_GATE)
    return launch_pwt_f16(loader, epi, a, st);
  return pw_dispatch<64>(loader, epi, a, st);
}

// Channels per workgroup: 64 (mu and s rows, 128 accumulator registers), which
// gives C / 64 workgroups per pixel tile.
// Prior head, quantiser and bits (Fig. 4 "Q", Supp. B.2) as the epilogue of
// the pointwise kernel: the head's rows are packed in passes of 32 mu rows
// followed by the 32 s rows of the same channels, so one workgroup holds both
// for its 128 latent pixels x 32 channels.  Bit partial sums: one per
// (tile, pass), reduced in a fixed order by k_reduce.
int prior_partials_f16(int C, int P) { return ((P + 127) / 128) * (C / 32); }

hipError_t launch_prior_f16(const PriorArgs& pa, hipStream_t st, int* n_partials) {
  if (pa.C % 32) return hipErrorInvalidValue;
  PwArgs a;
  std::memset(&a, 0, sizeof(a));
  a.wfrag = pa.wfrag;
  a.bias = pa.bias;
  a.K = pa.K ? pa.K : pa.C;
  a.N = pa.N ? pa.N : 2 * pa.C;
  a.ld0 = pa.ld0;
  a.c_off = pa.c_off;
  a.add = pa.add;
  a.add_ld = pa.add_ld;
  a.add_s = pa.add_s;
  a.add_c0 = pa.add_c0;
  a.add_f32 = pa.add_f32;
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
  a.k_out = pa.k_out;
  a.scales = pa.scales;
  if (n_partials) *n_partials = ((pa.P + 127) / 128) * (a.N / 64);
  return pw_dispatch<64>(LD_NHWC, pa.decode == 2 ? EP_SCALES : pa.decode ? EP_PRIOR_DEC : EP_PRIOR, a, st);
}

hipError_t launch_zquant_f16(const PwArgs& a, hipStream_t st, int* n_partials) {
  if (a.N != 64 || a.K % 64) return hipErrorInvalidValue;
  if (n_partials) *n_partials = (a.P + 127) / 128;
  return pw_dispatch<64>(LD_DOWN, EP_ZQUANT, a, st);
}

}  // namespace nc
