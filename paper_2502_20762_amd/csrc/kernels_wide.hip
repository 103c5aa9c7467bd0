// Depthwise 3x3 of a DC block as a kernel of its own, for the wide blocks
// (C > 256: the Large model's width, Supp. "Performance for a Large Model")
// whose weights and hidden layer do not fit the LDS of one CU in a fused
// block.  A wide block is three launches: this kernel, the pointwise C -> 2C
// with the LeakyReLU epilogue, the pointwise 2C -> C with the residual
// epilogue (Supp. B.1; Alg. 1 on the integer path).
//
// Bound by loads from L2.  A thread owns 8 channels of a strip of ROWS x COLS pixels: it
// loads its 9 x 8 weights once and every pixel of the strip's halo once (coalesced over
// the channel groups of a pixel), (ROWS + 2) (COLS + 2) / (ROWS COLS) 16-byte loads per
// output instead of nine, and an XCD takes a contiguous range of strips, so that its L2
// holds the halos.  fp16, 1080p, C = 512 (67 MB in and out): one thread per output pixel
// 38.6 us, strips of 4 x 1 30 us, 8 x 1 25, 4 x 2 22, 8 x 2 18.8 (3.6 TB/s), 4 x 4 28.
#include <type_traits>

#include "common.hpp"
#include "internal.hpp"

namespace nc {

// fp16: a = b + sum over (ky, kx) of w * z in fp32 (taps row by row, the
// order of the fused block), one rounding to fp16; taps outside the map are
// zero.  int16: a_i = clip(RHE((512 b + sum w_i z_i) / 8192)) in wrapping int32
// (Alg. 1; the sum is the same in any order).
template <bool IS_INT, int ROWS, int COLS>
__global__ __launch_bounds__(256) void k_dw3x3(const void* zv, const uint32_t* dww, void* outv, int C, int h, int w) {
  using T = std::conditional_t<IS_INT, int16_t, f16>;
  using V = std::conditional_t<IS_INT, shortx8, half8>;
  using A = std::conditional_t<IS_INT, int, float>;
  const T* const z = (const T*)zv;
  T* const out = (T*)outv;
  const int G = C / 8;
  const int64_t t = (int64_t)xcd_tile(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
  const int g = (int)(t % G);
  const int64_t strip = t / G;
  const int wc = (w + COLS - 1) / COLS;
  const int x0 = (int)(strip % wc) * COLS, y0 = (int)(strip / wc) * ROWS;
  if (y0 >= h) return;
  uint32_t wt[9][4];  // tap, channel pair
  A bias[8];
  if constexpr (IS_INT) {
    // 2 channel quads of 24 words: per tap the int16 pairs (c, c+1), (c+2, c+3), then the 4 biases 512 b
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uint32_t* q = dww + 24 * (2 * g + i);
      uint32_t v[24];
#pragma unroll
      for (int u = 0; u < 6; ++u) {
        const intx4 r = *(const intx4*)(q + 4 * u);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * u + e] = (uint32_t)r[e];
      }
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        wt[k][2 * i] = v[2 * k];
        wt[k][2 * i + 1] = v[2 * k + 1];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) bias[4 * i + e] = (int)v[18 + e];
    }
  } else {
    // 4 channel pairs of 12 words: 9 taps as fp16 pairs, the 2 biases (fp32), a pad word
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t* q = dww + 12 * (4 * g + i);
      uint32_t v[12];
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        const intx4 r = *(const intx4*)(q + 4 * u);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * u + e] = (uint32_t)r[e];
      }
#pragma unroll
      for (int k = 0; k < 9; ++k) wt[k][i] = v[k];
      bias[2 * i] = __builtin_bit_cast(float, v[9]);
      bias[2 * i + 1] = __builtin_bit_cast(float, v[10]);
    }
  }
  A acc[ROWS][COLS][8];
#pragma unroll
  for (int r = 0; r < ROWS + 2; ++r) {  // map row y0 - 1 + r
    const int yy = y0 - 1 + r;
    V v[COLS + 2];
#pragma unroll
    for (int kx = 0; kx < COLS + 2; ++kx) {
      const int xx = x0 + kx - 1;
      v[kx] = V{};
      if (yy >= 0 && yy < h && xx >= 0 && xx < w) v[kx] = *(const V*)(z + ((size_t)yy * w + xx) * C + 8 * g);
    }
    if (r < ROWS)
#pragma unroll
      for (int c = 0; c < COLS; ++c)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[r][c][e] = bias[e];
    // output row r - ky takes this row as its tap row ky
#pragma unroll
    for (int ky = 0; ky < 3; ++ky) {
      const int o = r - ky;
      if (o < 0 || o >= ROWS) continue;
#pragma unroll
      for (int k = 0; k < 3 * COLS; ++k)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int c = k / 3, kx = k % 3;
          A& sum = acc[o][c][e];
          const uint32_t pr = wt[3 * ky + kx][e >> 1];
          if constexpr (IS_INT) {
            const int wv = e & 1 ? (int)pr >> 16 : (int)(short)(pr & 0xFFFFu);
            sum = (int)((uint32_t)sum + (uint32_t)(wv * (int)v[c + kx][e]));
          } else {
            const half2 wv = __builtin_bit_cast(half2, pr);
            sum = fmaf((float)wv[e & 1], (float)v[c + kx][e], sum);
          }
        }
    }
    if (r >= 2 && y0 + r - 2 < h)
#pragma unroll
      for (int c = 0; c < COLS; ++c) {
        if (x0 + c >= w) continue;
        V o;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          if constexpr (IS_INT) o[e] = (short)rescale13(acc[r - 2][c][e]);
          else o[e] = (f16)acc[r - 2][c][e];
        }
        *(V*)(out + ((size_t)(y0 + r - 2) * w + x0 + c) * C + 8 * g) = o;
      }
  }
}

template <bool IS_INT>
static hipError_t launch_dw3x3(const void* src, const void* dww, void* dst, int C, int h, int w, hipStream_t st) {
  if (C % 8 || h <= 0 || w <= 0) return hipErrorInvalidValue;
  auto grid = [&](int rows, int cols) {
    const int64_t n = ((int64_t)((h + rows - 1) / rows) * ((w + cols - 1) / cols) * (C / 8) + 255) / 256;
    return dim3((unsigned)((n + 7) / 8 * 8));
  };
  // Strips of 8 x 2 while they still give every SIMD a wave (256 workgroups), of 2 x 1 while
  // these give more than 1.5 workgroups per CU, else single pixels.  us per decode with four
  // blocks, fp16 then int16:
  //   2 x 1 / 8 x 2 (workgroups of 8 x 2): 832 x 480 C = 512 (104) 178 / 190, 280 / 287; 720p C
  //     = 384 (184) 222 / 224, 391 / 388; C = 512 (240) 299 / 290, 539 / 522; 1080p C = 384
  //     (384) 388 / 361, 707 / 669; C = 512 (512) 553 / 498, 1103 / 1044
  //   1 x 1 / 2 x 1 (workgroups of 2 x 1), C = 512: 64 x 64 (8) 111 / 115, 184 / 188; 256 x 256
  //     (128) 115 / 118, 191 / 193; 320 x 480 (304) 127.5 / 130.5, 205.4 / 206.7; 384 x 512
  //     (384) 128.5 / 129.4, 203.9 / 204.1; 384 x 640 (480) 137.4 / 135.2, 212.6 / 208.0; 832 x
  //     480 (784) 178 / 175, 281 / 279
  if ((int64_t)grid(8, 2).x * 4 >= 1024)
    launch(k_dw3x3<IS_INT, 8, 2>, grid(8, 2), dim3(256), st, src, (const uint32_t*)dww, dst, C, h, w);
  else if (grid(2, 1).x > 384)
    launch(k_dw3x3<IS_INT, 2, 1>, grid(2, 1), dim3(256), st, src, (const uint32_t*)dww, dst, C, h, w);
  else
    launch(k_dw3x3<IS_INT, 1, 1>, grid(1, 1), dim3(256), st, src, (const uint32_t*)dww, dst, C, h, w);
  return hipGetLastError();
}

hipError_t launch_dw3x3_f16(const void* src, const void* dww, void* dst, int C, int h, int w, hipStream_t st) {
  return launch_dw3x3<false>(src, dww, dst, C, h, w, st);
}

hipError_t launch_dw3x3_i16(const void* src, const void* dww, void* dst, int C, int h, int w, hipStream_t st) {
  return launch_dw3x3<true>(src, dww, dst, C, h, w, st);
}

}  // namespace nc
