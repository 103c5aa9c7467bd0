// fp16 pointwise contractions with large register tiles: the two halves of a wide DC
// block (C > 256), from C = 128 on the folded input convs of both transforms
// (patch embed + fuse, upsample + fuse) and the reconstruction: out^T[rows][pixels] = W act^T + b.
//
// A workgroup of 4 waves, one per SIMD, computes 128 RT rows x 32 PG pixels: wave w the
// RT 32-row tiles from 32 RT w on, for all PG pixel groups.  The weight fragments
// come straight from L2 into registers as MFMA A operands, each feeding PG MFMAs, a
// whole stage (64 contraction indices) ahead; the activations of a stage arrive in
// LDS by direct global->LDS loads one stage ahead (two buffers).  At most 256
// registers per lane and 64 KiB of LDS leave room for two workgroups per CU: one's
// waits and stores run beside the other's MFMAs.  (One workgroup of 256 rows x 256
// pixels per CU, with 4 or with 8 waves, was slower: 50 and 44 us against 40 for
// K = 512, N = 1024 at 1080p.)  The sums are fp32; the results are rounded to fp16
// once, parked in LDS and stored as 16-byte vectors.
#include <type_traits>
#include <utility>

#include "common.hpp"
#include "internal.hpp"

namespace nc {

namespace {

template <int LOADER, int EPI, int RT, int PG, bool BIAS_FIRST>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_pwt_f16(PwArgs a) {
  constexpr int NR = 128 * RT, NPX = 32 * PG;  // rows and pixels of a workgroup
  constexpr int STAGE = NPX * 128;             // activation bytes of a stage
  constexpr int OUT = EPI == EP_GATE ? NR / 2 : NR;  // stored channels
  constexpr int PARK = NPX * OUT * 2;
  constexpr int SMEM = 2 * STAGE > PARK ? 2 * STAGE : PARK;
  __shared__ __attribute__((aligned(1024))) char smem[SMEM];
  static_assert(EPI != EP_GATE || RT == 2, "a wave holds h1 and h2 of its channels");
  const int ntile = (a.P + NPX - 1) / NPX, npass = a.N / NR;
  const int lin = xcd_tile(blockIdx.x, gridDim.x);
  const int tile = lin / npass;
  if (tile >= ntile) return;
  const int n0 = (lin - tile * npass) * NR;
  // the upsample that follows the prior in an encode: workgroup 0 first adds up
  // the frame's rate partials
  if constexpr (EPI == EP_UP)
    if (a.bits_out && blockIdx.x == 0) block_sum_to(a.sum_base, a.n_sum, a.bits_out);
  const int lane = threadIdx.x & 63, h = lane >> 5, n = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nk = a.K / 64;

  // activation stage kc into buffer b: instruction i = wave + 4 m, 16-byte unit S of
  // the stage: pixel S / 8, position S % 8 holds vector (S % 8) ^ ((pixel / 2) % 8)
  // (byte offsets fit 32 bits: an operand has at most 2^20 pixels x 2^10 channels)
  uint32_t ao[PG], ao1[PG];
#pragma unroll
  for (int m = 0; m < PG; ++m) {
    const int S = (wave + 4 * m) * 64 + lane, p = S >> 3, v = (S & 7) ^ ((p >> 1) & 7);
    const int gp = min(tile * NPX + p, a.P - 1);  // pixels past the end reload the last one
    if constexpr (LOADER == LD_FRAME_CTX) {
      // k = 64 c + 8 i + j < 192: colour c, frame row 8 py + i = 8 py + v, columns 8 px .. + 7; then the context
      const int py = gp / a.w8, px = gp - py * a.w8;
      ao[m] = 2u * ((uint32_t)(8 * py + v) * (uint32_t)a.W + 8u * (uint32_t)px);
      ao1[m] = 2u * (uint32_t)gp * (uint32_t)a.C1 + 16u * v;
    } else if constexpr (LOADER == LD_UP_CTX) {
      // k < C0: yhat at the 1/16 pixel; then the context at its child pixel of the pass's sub-position
      const int sp = n0 / a.Cdst, w16 = a.w8 >> 1;
      const int Y = gp / w16, X = gp - Y * w16;
      ao[m] = 2u * (uint32_t)gp * (uint32_t)a.C0 + 16u * v;
      ao1[m] = 2u * (uint32_t)((2 * Y + (sp >> 1)) * a.w8 + 2 * X + (sp & 1)) * (uint32_t)a.C1 + 16u * v;
    } else {
      ao[m] = 2u * (uint32_t)gp * (uint32_t)a.K + 16u * v;
    }
  }
  const int k1 = LOADER == LD_FRAME_CTX ? 3 : LOADER == LD_UP_CTX ? a.C0 / 64 : nk;  // first stage of the second operand
  auto load_act = [&](int kc, int b) __attribute__((always_inline)) {
    const bool second = LOADER != LD_NHWC && kc >= k1;
    const char* const base =
        second ? (const char*)a.src1 + 128 * (kc - k1)
               : (const char*)a.src0 + (LOADER == LD_FRAME_CTX ? 2 * (size_t)kc * a.H * a.W : (size_t)128 * kc);
#pragma unroll
    for (int m = 0; m < PG; ++m) dma16s(base, second ? ao1[m] : ao[m], smem + b * STAGE + (wave + 4 * m) * 1024);
  };
  const char* const wf = (const char*)a.wfrag + (size_t)(n0 / 32 + RT * wave) * (a.K / 16) * 1024;
  half8 qa[2][4][RT];
  auto load_w = [&](int kc, int b) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int t = 0; t < RT; ++t)
        qa[b][ks][t] = *(const half8*)(wf + ((size_t)t * (a.K / 16) + 4 * kc + ks) * 1024 + lane * 16);
  };
  // The sums of the model at C = 256 start at the bias, at other widths it comes last: the
  // order these layers have always had, so that a frame coded with one kernel has the
  // same values with another.  A bias that comes last is held from the start where the
  // registers allow (loaded at the end it costs 0.5 us of a 6 us launch).
  const float* const bp = (const float*)a.bias + n0 + 32 * RT * wave + 4 * h;
  constexpr bool HELD = BIAS_FIRST || RT * PG < 8;
  floatx4 bias[RT][4];
  auto load_bias = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int q = 0; q < 4; ++q) bias[t][q] = *(const floatx4*)(bp + 32 * t + 8 * q);
  };
  if constexpr (HELD) load_bias();
  floatx16 acc[RT][PG];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int g = 0; g < PG; ++g)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[t][g][i] = BIAS_FIRST ? bias[t][i / 4][i % 4] : 0.f;
  // B fragment of k-step ks, group g: pixel 32 g + n, vector 2 ks + h
  int bo[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) bo[ks] = n * 128 + (((2 * ks + h) ^ ((n >> 1) & 7)) << 4);
  // everything requested has arrived, for every wave
  auto arrive = [&]() __attribute__((always_inline)) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0), lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  load_act(0, 0);
  load_w(0, 0);
  auto stage = [&](int kc, auto bc) __attribute__((always_inline)) {
    constexpr int b = decltype(bc)::value;
    arrive();
    if (kc + 1 < nk) {
      load_w(kc + 1, 1 - b);
      load_act(kc + 1, 1 - b);
    }
    __builtin_amdgcn_sched_barrier(0);
    const char* const sb = smem + b * STAGE;
    half8 B[2][PG];
#pragma unroll
    for (int g = 0; g < PG; ++g) B[0][g] = *(const half8*)(sb + bo[0] + g * 4096);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      if (ks < 3) {
#pragma unroll
        for (int g = 0; g < PG; ++g) B[(ks + 1) & 1][g] = *(const half8*)(sb + bo[ks + 1] + g * 4096);
      }
#pragma unroll
      for (int g = 0; g < PG; ++g)
#pragma unroll
        for (int t = 0; t < RT; ++t) acc[t][g] = mfma_f16(qa[b][ks][t], B[ks & 1][g], acc[t][g]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  for (int kc = 0; kc < nk; kc += 2) {
    stage(kc, std::integral_constant<int, 0>{});
    if (kc + 1 < nk) stage(kc + 1, std::integral_constant<int, 1>{});
  }
  if constexpr (!BIAS_FIRST) {
    if constexpr (!HELD) load_bias();
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int g = 0; g < PG; ++g)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[t][g][i] += bias[t][i / 4][i % 4];
  }
  lds_barrier();  // every wave is done reading the stages

  // park: row = pixel (OUT channels), its 16-byte unit u at (u & ~15) | ((u ^ pixel) & 15)
  auto unit = [&](int p, int u) __attribute__((always_inline)) {
    return smem + p * (OUT * 2) + (((u & ~15) | ((u ^ p) & 15)) << 4);
  };
  if constexpr (EPI == EP_RESID) {
    // the residual tile first, then each lane adds its values in place
    for (int i = wave; i < PARK / 1024; i += 4) {
      const int S = i * 64 + lane, p = S / (OUT / 8), pos = S % (OUT / 8);
      const int u = (pos & ~15) | ((pos ^ p) & 15);
      const int gp = min(tile * NPX + p, a.P - 1);
      dma16((const f16*)a.res + (size_t)gp * a.Cdst + n0 + 8 * u, smem + i * 1024);
    }
    arrive();
  }
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    if (EPI == EP_GATE && t) break;
#pragma unroll
    for (int g = 0; g < PG; ++g) {
      const int p = 32 * g + n;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int cc = 32 * ((EPI == EP_GATE ? 1 : RT) * wave + t) + 8 * q + 4 * h;
        half4* const at = (half4*)(unit(p, cc >> 3) + 8 * h);
        half4 o;
        if constexpr (EPI == EP_RESID) {
          const half4 r = *at;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = (f16)(acc[t][g][4 * q + e] + (float)r[e]);
        } else if constexpr (EPI == EP_LRELU) {
          // as the fused block: the hidden value rounded to fp16, then max(h, 0.1 h) in fp16
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const f16 hv = (f16)acc[t][g][4 * q + e];
            o[e] = __builtin_fmaxf16(hv, hv * (f16)0.1f);
          }
        } else if constexpr (EPI == EP_GATE) {
          // as the fused gated block: WSiLU(h1) = h1 sigmoid(4 h1) rounded to fp16,
          // then g = WSiLU(h1) h2 rounded to fp16 (the packed pw1 rows: 32 h1, 32 h2)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float u = acc[0][g][4 * q + e];
            const f16 s1 = (f16)(u / (1.f + __expf(-4.f * u)));
            o[e] = (f16)((float)s1 * acc[1][g][4 * q + e]);
          }
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = (f16)acc[t][g][4 * q + e];
        }
        *at = o;
      }
    }
  }
  lds_barrier();
  if constexpr (EPI == EP_REC) {
    // rows 64 c + 8 i + j < 192: a 16-byte store covers the 8 frame pixels j of (colour
    // c, row i) of one 1/8-scale pixel; consecutive threads walk the pixels, clamped to
    // [0, 1] (the same as clamping before the rounding)
#pragma unroll 4
    for (int i = threadIdx.x; i < NPX * OUT / 8; i += 256) {
      const int p = i % NPX, gp = tile * NPX + p, u = n0 / 8 + i / NPX;
      if (gp >= a.P || u >= 24) continue;
      const half8 v = *(const half8*)unit(p, i / NPX);
      half8 o;
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = __builtin_fminf16(__builtin_fmaxf16(v[e], (f16)0.f), (f16)1.f);
      const int py = gp / a.w8, px = gp - py * a.w8;
      __builtin_nontemporal_store(
          o, (half8*)((f16*)a.dst + (size_t)(u >> 3) * a.H * a.W + (size_t)(8 * py + (u & 7)) * a.W + 8 * px));
    }
    return;
  }
  const int ch0 = EPI == EP_GATE ? n0 / 2 : n0;
#pragma unroll 4
  for (int i = threadIdx.x; i < NPX * OUT / 8; i += 256) {
    const int p = i / (OUT / 8), u = i % (OUT / 8);
    const int gp = tile * NPX + p;
    if (gp >= a.P) continue;
    size_t off;
    if constexpr (EPI == EP_UP) {  // rows n = sp C + c, all in one sub-position sp
      const int sp = n0 / a.Cdst, w16 = a.w8 >> 1;
      const int Y = gp / w16, X = gp - Y * w16;
      off = (size_t)((2 * Y + (sp >> 1)) * a.w8 + 2 * X + (sp & 1)) * a.Cdst + (n0 - sp * a.Cdst) + 8 * u;
    } else {
      off = (size_t)gp * a.Cdst + ch0 + 8 * u;
    }
    *(half8*)((f16*)a.dst + off) = *(const half8*)unit(p, u);
  }
}

template <int LOADER, int EPI, int RT, int PG>
hipError_t go(const PwArgs& a, int wgs, hipStream_t st) {
  const dim3 grid((wgs + 7) / 8 * 8);
  if constexpr (EPI == EP_REC || EPI == EP_UP || EPI == EP_NHWC) {
    if (EPI == EP_REC ? a.K == 256 : a.Cdst == 256) {
      launch(k_pwt_f16<LOADER, EPI, RT, PG, true>, grid, dim3(256), st, a);
      return hipGetLastError();
    }
  }
  launch(k_pwt_f16<LOADER, EPI, RT, PG, false>, grid, dim3(256), st, a);
  return hipGetLastError();
}

int wgs(const PwArgs& a, int rt, int pg) { return (a.P + 32 * pg - 1) / (32 * pg) * (a.N / (128 * rt)); }

// Tile (rows x pixels) by the number of workgroups, 128 RT x 32 PG: 256 x 128 where it
// gives enough of them, else 128 x 128, else 128 x 64 (more workgroups, each weight
// fragment feeding fewer MFMAs).  us, fp16, 256 x 128 / 128 x 128 / 128 x 64, "-" not
// dividing:
//   block halves, K = 512 N = 1024:   1080p 42.8 / 43.6 / -, 720p 21.9 / 22.9 / 24.2,
//     832 x 480 13.0 / 12.1 / 13.0, 96 x 96 11.3 / 7.9 / 7.1
//   K = 1024 N = 512:                 720p 24.8 / 23.1 / 25.1, 832 x 480 20.0 / 14.7 / 13.1
//   patch embed + fuse, K = 448 N = 256: 4K 47.7 / 55.1 / 65.2, 1080p 16.1 / 16.0 / 16.6,
//     720p 13.1 / 11.1 / 10.1
// which puts the line at 384 workgroups (1.5 per CU).  Upsample + fuse (its operand rows
// and stores lie two pixels apart), K = 512 N = 1024: 4K 61.7 / 67.1 / 63.7, 1080p 20.9 /
// 18.4 / 16.4, 720p 18.5 / 14.3 / 10.0; K = 1024 N = 2048: 1080p 52.7 / 70.9 / 57.7: the
// first from 512 workgroups on, else the last.  Reconstruction (N = 192 padded to 256),
// with 256 x 64 in the middle: K = 256 1080p 9.8 us against 12.8 with 128 x 64, 720p 7.2
// / 6.8, 832 x 480 6.6 / 5.6; K = 512 1080p 13.4 / 15.6.
// At 1080p, C = 512 the halves took 58 and 54 us with both operands staged through LDS,
// 39 and 40 us here (870 TFLOP/s; the same card).
template <int LOADER, int EPI>
hipError_t pick(const PwArgs& a, hipStream_t st) {
  constexpr bool up = EPI == EP_UP;
  const bool rows256 = a.N % 256 == 0 && (!up || a.Cdst % 256 == 0);
  if (rows256 && wgs(a, 2, 4) >= (up ? 512 : 384)) return go<LOADER, EPI, 2, 4>(a, wgs(a, 2, 4), st);
  if constexpr (EPI == EP_REC) {
    if (wgs(a, 2, 2) >= 384) return go<LOADER, EPI, 2, 2>(a, wgs(a, 2, 2), st);
  } else if constexpr (!up) {
    if (wgs(a, 1, 4) >= 384) return go<LOADER, EPI, 1, 4>(a, wgs(a, 1, 4), st);
  }
  return go<LOADER, EPI, 1, 2>(a, wgs(a, 1, 2), st);
}

}  // namespace

hipError_t launch_pwt_f16(int loader, int epi, const PwArgs& a, hipStream_t st) {
  if (a.K % 64 || a.ld0) return hipErrorInvalidValue;
  if (loader == LD_NHWC && epi == EP_REC && a.N == 192) {
    // its weight image and bias are padded with zeros to 256 rows
    PwArgs r = a;
    r.N = 256;
    return pick<LD_NHWC, EP_REC>(r, st);
  }
  if (a.N % 128 || (epi == EP_UP && a.Cdst % 128)) return hipErrorInvalidValue;
  if (loader == LD_NHWC && epi == EP_LRELU) return pick<LD_NHWC, EP_LRELU>(a, st);
  if (loader == LD_NHWC && epi == EP_RESID) return pick<LD_NHWC, EP_RESID>(a, st);
  if (loader == LD_FRAME_CTX && epi == EP_NHWC) return pick<LD_FRAME_CTX, EP_NHWC>(a, st);
  if (loader == LD_UP_CTX && epi == EP_UP) return pick<LD_UP_CTX, EP_UP>(a, st);
  if (loader == LD_NHWC && epi == EP_GATE && a.N % 256 == 0) {  // a wave needs h1 and h2 rows: 256-row passes
    if (wgs(a, 2, 4) >= 384) return go<LD_NHWC, EP_GATE, 2, 4>(a, wgs(a, 2, 4), st);
    return go<LD_NHWC, EP_GATE, 2, 2>(a, wgs(a, 2, 2), st);
  }
  return hipErrorInvalidValue;
}

}  // namespace nc
