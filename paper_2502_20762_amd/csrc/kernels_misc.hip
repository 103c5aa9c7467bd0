// Small kernels: deterministic bit reduction, the standalone rate estimate,
// zero fill, and state layout conversion (channels-last <-> planar).
#include "common.hpp"
#include "internal.hpp"

namespace nc {

// One workgroup; thread t sums partials t, t+256, ... in order, then a fixed
// LDS tree.  The result does not depend on timing.
__global__ __launch_bounds__(256) void k_reduce(const double* part, int n, double* out) {
  __shared__ double sh[256];
  double v = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) v += part[i];
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = sh[0];
}

// Block b owns elements [b*chunk, min(n, (b+1)*chunk)); chunk depends only on n.
// The scale of element i is sigma[i] (float32), or on the integer path
// sigma_tab[s[i] + 32768] for the prior's int16 scale output s (a table of
// max(softplus(s / 512), 0.11) over every int16 value).
template <bool INT_SCALE>
__global__ __launch_bounds__(256) void k_bits(const int16_t* q, const void* scale, const float* sigma_tab, int64_t n,
                                              int64_t chunk, double* part) {
  const int64_t lo = (int64_t)blockIdx.x * chunk;
  const int64_t hi = min(n, lo + chunk);
  double v = 0.0;
  for (int64_t i = lo + threadIdx.x; i < hi; i += 256) {
    float sg;
    if constexpr (INT_SCALE) sg = sigma_tab[(int)((const int16_t*)scale)[i] + 32768];
    else sg = ((const float*)scale)[i];
    v += (double)symbol_bits((float)q[i], sg);
  }
  __shared__ double red[4];
  v = wave_sum(v);
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) red[wave] = v;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = ((red[0] + red[1]) + red[2]) + red[3];
}

// Zeroes two ranges of 16-byte units (the two tensors of a context's state).  Bound by
// launch and memory: both state tensors of a 1080p frame (21 MB) took 10.2 + 5.1 us as two
// launches of 4-byte stores, 10.0 here (2,048 workgroups; 512 12.9 us, 1,024 10.8, one store per
// thread 13.4, non-temporal 9.2 but the kernels that read the state next lose more).
__global__ __launch_bounds__(256) void k_fill_zero(intx4* p0, size_t n0, intx4* p1, size_t n1) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n0 + n1; i += (size_t)gridDim.x * 256)
    (i < n0 ? p0[i] : p1[i - n0]) = intx4{};
}

// State layout conversion, planar[c*P + p] <-> nhwc[p*C + c] (2-byte elements),
// bound by memory.  A workgroup turns one tile of 64 channels x 64 pixels
// through LDS, so that both sides move whole lines: 128 bytes of a pixel's
// channels, 128 bytes of a channel's pixels (16 bytes per lane where the rows
// are 16-byte aligned: P a multiple of 8 and an aligned buffer).  C is a
// multiple of 64.  Element by element (each lane striding through the other
// layout) the context feature of a 1080p frame (16.7 MB each way) took 58 us
// in and 87 us out, the tiles take 7.8 us (4.3 TB/s), 8.2 us with the latent's 4.2 MB in the
// same launch (13.1 as two); at 4K 490 against 25 us.
constexpr int kTrLd = 64 + 2;  // LDS row stride (elements): rows one bank apart

struct StateCopy {
  const uint16_t* src;
  uint16_t* dst;
  int P, tiles;  // pixels, 64-pixel tiles
};

// Both tensors of the state in one launch (a NULL tensor has no tiles).
template <bool TO_PLANAR>
__global__ __launch_bounds__(256) void k_transpose(StateCopy s0, StateCopy s1, int C) {
  __shared__ uint32_t tile32[64 * kTrLd / 2];
  uint16_t* const tile = (uint16_t*)tile32;  // [channel][pixel]
  const bool second = (int)blockIdx.x >= s0.tiles;
  const uint16_t* const src = second ? s1.src : s0.src;
  uint16_t* const dst = second ? s1.dst : s0.dst;
  const int P = second ? s1.P : s0.P;
  const int p0 = ((int)blockIdx.x - (second ? s0.tiles : 0)) * 64, c0 = blockIdx.y * 64;
  const int np = min(64, P - p0);
  const bool vec = P % 8 == 0 && (uintptr_t)(TO_PLANAR ? dst : src) % 16 == 0;
  // one 16-byte vector per step: NHWC: 8 channels of pixel i / 8; planar: 8 pixels of channel i / 8
  auto nhwc_at = [&](int i) { return (size_t)(p0 + (i >> 3)) * C + c0 + 8 * (i & 7); };
  auto planar_at = [&](int i) { return (size_t)(c0 + (i >> 3)) * P + p0 + 8 * (i & 7); };
  const int t = threadIdx.x;
  if constexpr (TO_PLANAR) {
    shortx8 v[2] = {};
#pragma unroll
    for (int j = 0; j < 2; ++j)
      if (((t + 256 * j) >> 3) < np) v[j] = *(const shortx8*)(src + nhwc_at(t + 256 * j));
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 8; ++e) tile[(8 * (t & 7) + e) * kTrLd + ((t + 256 * j) >> 3)] = (uint16_t)v[j][e];
  } else {
    const int px = 8 * (t & 7);
    intx4 v[2] = {};
    const bool whole = vec && px + 8 <= np;
#pragma unroll
    for (int j = 0; j < 2; ++j)
      if (whole) v[j] = *(const intx4*)(src + planar_at(t + 256 * j));
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int i = t + 256 * j;
      uint16_t* row = tile + (i >> 3) * kTrLd + px;
      if (whole) {
#pragma unroll
        for (int e = 0; e < 4; ++e) ((uint32_t*)row)[e] = (uint32_t)v[j][e];
      } else {
        for (int e = 0; e < 8 && px + e < np; ++e) row[e] = src[planar_at(i) + e];
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int i = t + 256 * j;
    if constexpr (TO_PLANAR) {
      const int px = 8 * (i & 7);
      const uint16_t* row = tile + (i >> 3) * kTrLd + px;
      if (vec && px + 8 <= np) {
        intx4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (int)((const uint32_t*)row)[e];
        *(intx4*)(dst + planar_at(i)) = v;
      } else {
        for (int e = 0; e < 8 && px + e < np; ++e) dst[planar_at(i) + e] = row[e];
      }
    } else if ((i >> 3) < np) {
      shortx8 v;
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = (short)tile[(8 * (i & 7) + e) * kTrLd + (i >> 3)];
      *(shortx8*)(dst + nhwc_at(i)) = v;
    }
  }
}

// One workgroup per (64-pixel, 32-channel) tile: the planar symbols of the
// tile are staged through LDS (coalesced row reads), then each thread forms
// 8 consecutive channels of one pixel and stores them as one 16-byte vector.
// Channels c < C of q (planar, C x P) go to channel c_off + c of mu and yhat
// (NHWC, row stride ld); a NULL mu is zero.
template <bool IS_INT>
__global__ __launch_bounds__(256) void k_yhat_from_q(const int16_t* q, const void* mu, void* yhat, int C, int P, int ld,
                                                     int c_off) {
  __shared__ int16_t qs[32][64 + 2];
  const int ntp = (P + 63) / 64;
  const int tp = blockIdx.x % ntp, tc = blockIdx.x / ntp;
  const int p0 = tp * 64, c0 = tc * 32;
  for (int i = threadIdx.x; i < 32 * 64; i += 256) {
    const int cc = i >> 6, pp = i & 63;
    qs[cc][pp] = p0 + pp < P ? q[(size_t)(c0 + cc) * P + p0 + pp] : (int16_t)0;
  }
  __syncthreads();
  const int pp = threadIdx.x >> 2, g8 = threadIdx.x & 3;
  const int gp = p0 + pp;
  if (gp >= P) return;
  const size_t off = (size_t)gp * ld + c_off + c0 + 8 * g8;
  if constexpr (IS_INT) {
    shortx8 m = {};
    if (mu) m = *(const shortx8*)((const int16_t*)mu + off);
    shortx8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (short)clip16(512 * (int)qs[8 * g8 + e][pp] + (int)m[e]);
    *(shortx8*)((int16_t*)yhat + off) = o;
  } else {
    floatx4 m0 = {}, m1 = {};
    if (mu) {
      m0 = *(const floatx4*)((const float*)mu + off);
      m1 = *(const floatx4*)((const float*)mu + off + 4);
    }
    half8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (f16)((float)qs[8 * g8 + e][pp] + (e < 4 ? m0[e] : m1[e - 4]));
    *(half8*)((f16*)yhat + off) = o;
  }
}

hipError_t launch_yhat_from_q(const int16_t* q, const void* mu, void* yhat, int C, int P, bool is_int,
                              hipStream_t st, int ld, int c_off) {
  if (C % 32 || c_off % 8) return hipErrorInvalidValue;
  if (!ld) ld = C;
  const dim3 grid(((P + 63) / 64) * (C / 32));
  if (is_int) launch(k_yhat_from_q<true>, grid, dim3(256), st, q, mu, yhat, C, P, ld, c_off);
  else launch(k_yhat_from_q<false>, grid, dim3(256), st, q, mu, yhat, C, P, ld, c_off);
  return hipGetLastError();
}

hipError_t launch_reduce(const double* partials, int n, double* out, hipStream_t st) {
  launch(k_reduce, dim3(1), dim3(256), st, partials, n, out);
  return hipGetLastError();
}

hipError_t launch_estimate_bits(const int16_t* q, const void* scale, const float* sigma_tab, int64_t n,
                                double* partials, double* out, hipStream_t st) {
  const int64_t chunk = n > 0 ? (n + kBitsBlocks - 1) / kBitsBlocks : 1;
  if (sigma_tab)
    launch(k_bits<true>, dim3(kBitsBlocks), dim3(256), st, q, scale, sigma_tab, n, chunk, partials);
  else
    launch(k_bits<false>, dim3(kBitsBlocks), dim3(256), st, q, scale, sigma_tab, n, chunk, partials);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_reduce(partials, kBitsBlocks, out, st);
}

hipError_t launch_fill_zero(void* p0, size_t bytes0, void* p1, size_t bytes1, hipStream_t st) {
  if (bytes0 % 16 || bytes1 % 16) return hipErrorInvalidValue;
  const size_t n0 = bytes0 / 16, n1 = bytes1 / 16;
  if (n0 + n1 == 0) return hipSuccess;
  const int blocks = (int)std::min<size_t>((n0 + n1 + 255) / 256, 2048);
  launch(k_fill_zero, dim3(blocks), dim3(256), st, (intx4*)p0, n0, (intx4*)p1, n1);
  return hipGetLastError();
}

template <bool TO_PLANAR>
static hipError_t launch_transpose(const void* f_src, void* f_dst, int Pf, const void* y_src, void* y_dst, int Py, int C,
                                   hipStream_t st) {
  if (C % 64) return hipErrorInvalidValue;
  auto one = [](const void* s, void* d, int P) {
    return StateCopy{(const uint16_t*)s, (uint16_t*)d, P, s && d ? (P + 63) / 64 : 0};
  };
  const StateCopy f = one(f_src, f_dst, Pf), y = one(y_src, y_dst, Py);
  if (f.tiles + y.tiles == 0) return hipSuccess;
  launch(k_transpose<TO_PLANAR>, dim3(f.tiles + y.tiles, C / 64), dim3(256), st, f, y, C);
  return hipGetLastError();
}

hipError_t launch_state_to_planar(const void* f_src, void* f_dst, int Pf, const void* y_src, void* y_dst, int Py, int C,
                                  hipStream_t st) {
  return launch_transpose<true>(f_src, f_dst, Pf, y_src, y_dst, Py, C, st);
}

hipError_t launch_state_to_nhwc(const void* f_src, void* f_dst, int Pf, const void* y_src, void* y_dst, int Py, int C,
                                hipStream_t st) {
  return launch_transpose<false>(f_src, f_dst, Pf, y_src, y_dst, Py, C, st);
}

}  // namespace nc
