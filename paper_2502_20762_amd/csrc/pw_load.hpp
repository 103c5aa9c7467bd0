// Activation loads of the staged pointwise kernels (k_pw_f16, k_pw_i16): both hold 16-bit
// values in the same layouts, 128 pixels x 64 contraction indices per stage, loaded by
// 8 waves with two 16-byte global->LDS loads per lane.
#pragma once

#include "common.hpp"
#include "internal.hpp"

namespace nc {

// Everything that depends on the pixel (two integer divisions) is formed once, as
// 32-bit byte offsets (an operand has at most 2^20 pixels x 2^10 channels), and a stage
// only moves the wave-uniform base.  Forming a 64-bit address per load and stage, for the 2x2
// windows with a division by the channel count, cost 3 to 12 % of these short
// kernels, which issue few MFMAs per stage (us, before -> now): 2x2 down-convolution
// K = 1024 int16 1080p 18.0 -> 16.3, tiny 5.9 -> 5.2; upsample int16 20.4 -> 19.1;
// 64 x 64 fp16 upsample + fuse 3.7 -> 3.1.
template <int LOADER>
struct PwAct {
  uint32_t o0[2], o1[2];
  int tap = 0, kin = 0;  // LD_DOWN: the next stage's window tap and its first channel

  __device__ __forceinline__ void init(const PwArgs& a, int tile, int n0, int wave, int lane) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int px = (wave + 8 * i) * 8 + (lane >> 3), v = (lane & 7) ^ ((px >> 1) & 7);
      const uint32_t gp = (uint32_t)min(tile * 128 + px, a.P - 1);  // pixels past the end reload the last one
      if constexpr (LOADER == LD_NHWC) {
        o0[i] = 2u * gp * (uint32_t)(a.ld0 ? a.ld0 : a.C0) + 16u * v;
        o1[i] = 2u * gp * (uint32_t)a.C1 + 16u * v;
      } else if constexpr (LOADER == LD_FRAME || LOADER == LD_FRAME_CTX) {
        // unshuffle x8: k = 64 c + 8 i + j -> colour c = kc, frame row 8 py + i = 8 py + v, columns 8 px .. +7
        const uint32_t py = gp / (uint32_t)a.w8, x = gp - py * (uint32_t)a.w8;
        o0[i] = 2u * ((8u * py + v) * (uint32_t)a.W + 8u * x);
        o1[i] = LOADER == LD_FRAME_CTX ? 2u * gp * (uint32_t)a.C1 + 16u * v : 0u;
      } else {
        const uint32_t w16 = (uint32_t)a.w8 >> 1;
        const uint32_t Y = gp / w16, X = gp - Y * w16;
        if constexpr (LOADER == LD_UP_CTX) {
          const uint32_t sp = (uint32_t)(n0 / a.Cdst);
          o0[i] = 2u * gp * (uint32_t)a.C0 + 16u * v;
          o1[i] = 2u * ((2 * Y + (sp >> 1)) * (uint32_t)a.w8 + 2 * X + (sp & 1)) * (uint32_t)a.C1 + 16u * v;
        } else {
          // 2x2 stride 2: k = (2 i + j) Csrc + c from pixel (2 Y + i, 2 X + j)
          o0[i] = 2u * (2 * Y * (uint32_t)a.w8 + 2 * X) * (uint32_t)a.Csrc + 16u * v;
          o1[i] = 0;
        }
      }
    }
  }

  // stages must be requested in order, 0, 1, ..
  __device__ __forceinline__ void issue(const PwArgs& a, int kc, char* stage, int wave) {
    bool second = false;
    const char* base = (const char*)a.src0;
    if constexpr (LOADER == LD_FRAME) {
      base += 2 * (size_t)kc * a.H * a.W;
    } else if constexpr (LOADER == LD_FRAME_CTX) {
      second = kc >= 3;
      base = second ? (const char*)a.src1 + 128 * (kc - 3) : base + 2 * (size_t)kc * a.H * a.W;
    } else if constexpr (LOADER == LD_DOWN) {
      base += 2 * ((size_t)((tap >> 1) * a.w8 + (tap & 1)) * a.Csrc + kin);
      kin += 64;
      if (kin == a.Csrc) {
        kin = 0;
        ++tap;
      }
    } else {
      second = 64 * kc >= a.C0;
      base = second ? (const char*)a.src1 + 2 * (64 * kc - a.C0) : base + 128 * kc;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uint32_t first = o0[i], other = o1[i];  // values: a choice between the members would put them in memory
      dma16s(base, second ? other : first, stage + (wave + 8 * i) * 1024);
    }
  }
};

}  // namespace nc
