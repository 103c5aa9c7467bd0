// fp16 DC block (Supp. B.1, LeakyReLU and gated forms), C = 64, 128 and 256, on
// 8 x 8 pixel tiles, one block per launch or a chain of blocks.
//
// A workgroup of 4 waves owns one tile of 64 pixels (two 32-pixel MFMA
// groups), in at most 80 KiB of LDS and 256 registers per lane, so that two
// workgroups share a CU: one tile's VALU and memory phases (depthwise,
// hand-offs, ring exchange, stores) run beside the other's MFMA loops.
//   1. Depthwise.  The channels are split into groups of 64 (C / 64 of
//      them); each group's halo band (10 x 10 pixels, 128 bytes per pixel)
//      lies in a region of its own.  256 / C waves share a group, each
//      filtering its rows; lane = (channel pair, column half), accumulated in
//      fp32 from the bias (C = 256: v_dot2_f32_f16, below it an fma per tap),
//      rounded to fp16 once and kept in registers until the band has been read (the residual of the
//      wave's outputs, the band's interior, goes to registers too), then
//      written over the band as B fragments of a.
//   2. pw1.  The 2C hidden channels are chunks of 32; the waves run the chains
//      of their chunks over both pixel groups, the LeakyReLU (C = 256: on the
//      fp16-rounded value, below it in fp32) or the gate, and write the result
//      as pw2 B fragments.  C = 256 takes two rounds (the second writes over a).
//   3. pw2.  Each wave accumulates its 32-row output tiles from the bias over
//      the hidden layer; the residual enters through identity MFMAs (exact
//      products), at C = 256 before the hidden layer, below it after; the
//      sums are rounded to fp16 once.
// Where C = 256 and the smaller widths differ, each has the order and the roundings that its
// frames have always had, so that a stream does not depend on the kernel that coded it.
// Every weight fragment is read straight from global memory (L2) as an MFMA A
// operand and feeds both pixel groups.
#include <utility>

#include "common.hpp"
#include "dc_chain.hpp"
#include "internal.hpp"

namespace nc {

namespace {

constexpr int TH = 8, TW = 8;              // tile rows x columns at 1/8 scale
constexpr int BH = TH + 2, BW = TW + 2;    // halo band
constexpr int BROW = BW * 128;             // bytes of a band row (64 channels)
constexpr int XF = 1024 + 16;              // LDS stride of one B fragment
constexpr int BAND_INSTR = (BH * BW * 8 + 63) / 64;  // 13 direct loads of 1 KiB per band
constexpr int REG = BAND_INSTR * 1024;     // a 64-channel group's region: its band, later 8 fragments of a and 4 more
static_assert(12 * XF <= REG - 16 && BH * BW * 128 <= REG - 16, "twelve fragments per region, or a band, and the chains' word");

// Position swizzle of the 16-byte units of band pixel (row y, column x): with
// it the residual reads (16 lanes = two rows of 8 columns, one unit) and the
// fills fall in different LDS banks.
__device__ __forceinline__ constexpr int usw(int y, int x) { return ((x >> 1) & 3) | ((y & 1) << 2); }
// Position of lane slot L (pixel 8 r + x of its group of 4 rows, k half
// kh = L / 32) inside a 1 KiB B fragment, free of LDS bank conflicts both for
// the operand reads (16 consecutive lanes: a bijection mod 16) and for the
// depthwise's 4-byte writes (at one step: columns x and 7 - x, both k halves,
// four consecutive fragments, 65 units apart).
__device__ __forceinline__ constexpr int bslot(int L) {
  const int r = (L >> 3) & 3, x = L & 7, kh = L >> 5;
  const int kk = x < 4 ? x : 7 - x, side = x >> 2;
  return 16 * ((r >> 1) + 2 * kh) + 4 * ((side + 2 * (r & 1) + 2 * kh) & 3) + kk;
}

// How a width's work is laid over the four waves.
template <int C, bool GATED>
struct Geo {
  static constexpr int KS = C / 16;                 // pw1 k-steps
  static constexpr int FR = KS + 1 + 2 * (C / 32);  // fragments per hidden chunk in the weight image
  static constexpr int NG = C / 64;                 // channel groups
  static constexpr int RW = 4 / NG;                 // waves that share a channel group
  static constexpr int RPW = TH / RW;               // output rows per wave
  static constexpr int R = C == 256 ? 2 : 1;        // pw1 rounds
  static constexpr int C1 = C == 64 && !GATED ? 1 : 2;  // pw1 chunks per wave and round
  static constexpr int G1 = C == 64 && GATED ? 1 : 2;   // pixel groups of a wave's pw1
  static constexpr int T2 = C == 256 ? 2 : 1;       // pw2 output tiles per wave
  static constexpr int G2 = C == 64 ? 1 : 2;        // pixel groups of a wave's pw2
  static constexpr int K2 = (GATED ? C : 2 * C) / 16;  // pw2 k-steps
  static constexpr int KH = K2 / R;                 // of them per round
  static constexpr int N1 = R * KS;                 // weight-stream steps of pw1
  static constexpr int NT = N1 + K2;
  // LDS: the regions, fragments of the hidden layer that do not fit there, biases
  static constexpr int OX = NG * REG;
  static constexpr int NX = C == 256 ? (GATED ? 0 : 16) : 2 * KH;
  static constexpr int OBIAS = OX + NX * XF;
  static constexpr int SMEM = OBIAS + 12 * C;
  static constexpr int SYNC = REG - 16;  // a word no one else uses once the first band is in
  // registers per lane allow 2 workgroups per CU (4 at C = 64)
  static constexpr int WPE = C == 64 ? 4 : 2;
  static_assert(SMEM * WPE <= 160 * 1024, "WPE workgroups fit the LDS of a CU");

  // a's fragment (pixel group g, k-step s)
  static __device__ __forceinline__ constexpr int a_off(int g, int s) {
    return (s >> 2) * REG + (4 * g + (s & 3)) * XF;
  }
  // hidden fragment (g, k-step k) of round 0
  static __device__ __forceinline__ constexpr int h0_off(int g, int k) {
    if (C < 256) return OX + (2 * k + g) * XF;
    if (GATED) return (k >> 1) * REG + (8 + 2 * (k & 1) + g) * XF;
    return (k & 3) < 2 ? (k >> 2) * REG + (8 + 2 * (k & 3) + g) * XF : OX + (4 * (k >> 2) + 2 * ((k & 3) - 2) + g) * XF;
  }
  // ... of round 1 (C = 256), over a
  static __device__ __forceinline__ constexpr int h1_off(int g, int k) {
    return GATED ? (k >> 1) * REG + (2 * (k & 1) + g) * XF : a_off(g, k);
  }
};

template <typename F, int... T>
__device__ __forceinline__ void unrolled(F& f, std::integer_sequence<int, T...>) {
  (f(std::integral_constant<int, T>{}), ...);
}

// The 2x2 stride-2 downsample of a tile's last block output (C = 256), which
// lies in the interior of the bands: output rows 64 w .. + 63 (tiles c = 0, 1)
// of the tile's 16 latent pixels (4 x 4 at 1/16; columns 16 .. 31 of the MFMA
// repeat them), K = 4C with k = (2 i + j) C + c from pixel (2 Y + i, 2 X + j)
// (Fig. 4's downsampling to 1/16), the k-steps in order from zero, then the
// fp32 bias and one rounding to fp16: the arithmetic of the downsample launch,
// so the result is the same bit for bit.
__device__ __forceinline__ void dc64_down(const char* smem, const DcChainArgs& ca, const BlockArgs& a, int ty0, int tx0,
                                          int wave, int lane) {
  constexpr int C = 256, DK = 4 * C / 16;  // 64 k-steps
  const int h = lane >> 5, n = lane & 15, ly = n >> 2, lx = n & 3;
  const half8* wimg = (const half8*)ca.down_w + lane;  // fragment (row tile mt, k-step s) at [(mt DK + s) 64]
  auto afrag = [&](int s, int c) __attribute__((always_inline)) {
    return wimg[((size_t)(2 * wave + c) * DK + s) * 64];
  };
  // B of k-step s: channels 16 (s % 16) + 8 h .. + 7 of tap s / 16
  auto bfrag = [&](int s) __attribute__((always_inline)) {
    const int tap = s >> 4, y = 1 + 2 * ly + (tap >> 1), x = 1 + 2 * lx + (tap & 1);
    return *(const half8*)(smem + ((s & 15) >> 2) * REG + y * BROW + x * 128 + (((2 * (s & 3) + h) ^ usw(y, x)) << 4));
  };
  constexpr int PD = 8;  // prefetch distance (k-steps) of the weight fragments
  half8 qa[PD][2];
#pragma unroll
  for (int s = 0; s < PD; ++s)
#pragma unroll
    for (int c = 0; c < 2; ++c) qa[s][c] = afrag(s, c);
  floatx16 acc[2] = {floatx16{}, floatx16{}};
#pragma unroll
  for (int s = 0; s < DK; ++s) {
    const half8 B = bfrag(s);
    half8 A[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      A[c] = qa[s % PD][c];
      if (s + PD < DK) qa[s % PD][c] = afrag(s + PD, c);
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) acc[c] = mfma_f16(A[c], B, acc[c]);
  }
  // latent pixel (Y, X) lies in the image when its top-left child does (the
  // 1/8 sizes are even)
  const int Y = (ty0 >> 1) + ly, X = (tx0 >> 1) + lx;
  if ((lane & 31) < 16 && 2 * Y < a.h && 2 * X < a.w) {
    f16* y = (f16*)ca.down_y + (size_t)(Y * (a.w >> 1) + X) * C;
    const float* bias = (const float*)ca.down_b;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int ch = 64 * wave + 32 * c + 8 * q + 4 * h;
        const floatx4 bv = *(const floatx4*)(bias + ch);
        half4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (f16)(acc[c][4 * q + e] + bv[e]);
        *(half4*)(y + ch) = o;
      }
  }
}

// One block of a tile (FIRST: its band comes whole from a.src; LAST: its
// output goes whole to a.dst, or with ca->down_w set, and down, through the downsample
// to ca->down_y; otherwise the chain's ring and edge exchange).
template <int C, bool GATED, bool FIRST, bool LAST>
__device__ __forceinline__ bool dc64_block(char* smem, const BlockArgs& a, int b, int tile, int tiles_x, int tiles_y,
                                           int wave0, ChainRun& run, const DcChainArgs* ca, bool down = true) {
  using G = Geo<C, GATED>;
  constexpr int KS = G::KS, FR = G::FR, NT = G::NT, N1 = G::N1, KH = G::KH;
  const int tyi = tile / tiles_x, txi = tile - tyi * tiles_x;
  const int ty0 = tyi * TH, tx0 = txi * TW;
  // the wave and lane index, opaque to the compiler: keeps the per-step
  // offsets from being hoisted out of the chain's block loop, where they
  // would all stay live at once
  int wave = wave0;
  asm volatile("" : "+s"(wave));
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  const int h = lane >> 5;
  const int myslot = bslot(lane) * 16;
  const int lane16 = lane * 16;
  const f16* z = (const f16*)a.src;
  const f16* zpad = (const f16*)a.zpad;
  const char* w1 = (const char*)a.w1;
  // entry (hidden chunk) of the wave's chain c in round r, its pw2 tile t, its pixel groups
  const int pair0 = C == 64 ? wave >> 1 : wave;
  auto entry = [&](int r, int c) __attribute__((always_inline)) {
    if (GATED) return 2 * (4 * r + pair0) + c;
    return C == 64 ? wave : 8 * r + 2 * wave + c;
  };
  const int tile0 = C == 256 ? 2 * wave : C == 128 ? wave : wave >> 1;
  const int g1 = G::G1 == 1 ? wave & 1 : 0, g2 = G::G2 == 1 ? wave & 1 : 0;
  // fragment c of weight-stream step t
  auto afrag = [&](int t, int c) __attribute__((always_inline)) {
    int f;
    if (t < N1) {
      f = entry(t / KS, c) * FR + t % KS;
    } else {
      const int k = t - N1;
      f = (GATED ? 2 * (k >> 1) + 1 : k >> 1) * FR + KS + 1 + 2 * (tile0 + c) + (k & 1);
    }
    return *(const half8*)(w1 + (size_t)f * 1024 + lane16);
  };
  // of the two tiles on a CU, one leads in even blocks, the other in odd ones
  if constexpr (!(FIRST && LAST)) {
    if ((b ^ (blockIdx.x >> 8)) & 1) __builtin_amdgcn_s_setprio(1);
    else __builtin_amdgcn_s_setprio(0);
  }
  constexpr int PA = 4, PB = 2;  // prefetch distances (steps) of the A and B windows
  half8 qa[PA][2];
  auto nfrag = [](int t) constexpr { return t < N1 ? G::C1 : G::T2; };

  // ---- 1. depthwise: channel group cg, rows r0 .. r0 + RPW - 1
  half8 res[G::T2][G::G2][2];  // residual: (output tile, group, half q) B operands
  {
    const int cg = G::RW == 1 ? wave : wave / G::RW;
    const int r0 = G::RW == 1 ? 0 : (wave % G::RW) * G::RPW;
    const int cp = lane & 31, half = lane >> 5;
    half2 wt[9];
    float bias0, bias1;
    {
      const intx4* wsrc = (const intx4*)a.dww + 3 * (32 * cg + cp);
      intx4 q0 = wsrc[0], q1 = wsrc[1];
      intx3 q2 = *(const intx3*)(wsrc + 2);
      // consumed here, before the other loads are issued, so that the
      // compiler's wait for them does not also wait for those loads
      asm volatile("" : "+v"(q0), "+v"(q1), "+v"(q2));
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int x0 = q0[i], x1 = q1[i];
        wt[i] = __builtin_bit_cast(half2, x0);
        wt[4 + i] = __builtin_bit_cast(half2, x1);
      }
      const int x8 = q2[0], xb0 = q2[1], xb1 = q2[2];
      wt[8] = __builtin_bit_cast(half2, x8);
      bias0 = __builtin_bit_cast(float, xb0);
      bias1 = __builtin_bit_cast(float, xb1);
    }
    char* const band = smem + cg * REG;
    if constexpr (FIRST) {
      // the band by direct loads, split over the group's waves
#pragma unroll
      for (int i = 0; i < (BAND_INSTR + G::RW - 1) / G::RW; ++i) {
        const int ii = G::RW == 1 ? i : i * G::RW + wave % G::RW;
        if (ii < BAND_INSTR) {
          const int S = ii * 64 + lane;  // band unit: pixel S / 8, position S % 8
          const int bp = S >> 3, u = S & 7;
          const int by = bp / BW, bx = bp - by * BW;
          const int hy = ty0 - 1 + by, hx = tx0 - 1 + bx;
          const bool in = bp < BH * BW && hy >= 0 && hy < a.h && hx >= 0 && hx < a.w;
          dma16(in ? z + (size_t)(hy * a.w + hx) * C + 64 * cg + 8 * (u ^ usw(by, bx)) : zpad, band + ii * 1024);
        }
      }
    }
    // the block's biases (pw1 2C, pw2 C, fp32), through registers
    floatx4 bv = {};
    const int bi = wave * 64 + lane;
    if (bi < 3 * C / 4) bv = bi < C / 2 ? ((const floatx4*)a.b1)[bi] : ((const floatx4*)a.b2)[bi - C / 2];
    // the first weight fragments
#pragma unroll
    for (int s = 0; s < PA; ++s)
#pragma unroll
      for (int c = 0; c < 2; ++c)
        if (c < nfrag(s)) qa[s][c] = afrag(s, c);
    // The lane's outputs k = 0 .. 3 of a row, at tile column x(k), and its band reads.
    // C < 256: x = k + 4 half, six consecutive columns, the nine taps of an output row by row
    // and left to right (fp32 fma).
    // C = 256: the taps of a row are two dot2 pairs, (first, middle) and (0, last); the sums
    // of the 8 x 16 tiles' kernel run from the left in the left half of a 16-column group and
    // from the right in its right half, so here a tile at an even tile column runs from the
    // left (dir = 0) and the others from the right, and a frame has the same values on
    // either tile.  k = 0 is the column next to the ring (0 or 7), which is known last, k = 1 .. 3
    // the three others in that direction: role 0 (the half the direction starts from) x(k) = 0
    // .. 3 from its side, role 1 the far column first.
    constexpr bool DOT2 = C == 256;
    const int dir = txi & 1, role = half ^ dir;
    auto band_off = [&](int col) __attribute__((always_inline)) {
      return r0 * BROW + col * 128 + (((cp >> 2) ^ usw(0, col)) << 4) + (cp & 3) * 4;
    };
    // columns of k >= 1 (DOT2: lane order 1 .. 5) or of all outputs (0 .. 5); rows of odd index at va ^ 64
    int va[TW / 2 + 2];
#pragma unroll
    for (int i = 0; i < TW / 2 + 2; ++i) {
      const int from = role ? 3 + i : i;  // counted from the side the direction starts at
      va[i] = band_off(DOT2 ? (dir ? BW - 1 - from : from) : 4 * half + i);
    }
    int ve[3];  // DOT2: the columns of k = 0
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const int from = role ? 7 + j : j;
      ve[j] = band_off(dir ? BW - 1 - from : from);
    }
    // taps of a row as dot2 pairs in the lane's column order
    half2 W0a[3], W0b[3], W1a[3], W1b[3];
#pragma unroll
    for (int ky = 0; ky < 3; ++ky) {
      const half2 l = dir ? wt[3 * ky + 2] : wt[3 * ky], m = wt[3 * ky + 1], r = dir ? wt[3 * ky] : wt[3 * ky + 2];
      W0a[ky] = half2{l[0], m[0]};
      W0b[ky] = half2{(f16)0.f, r[0]};
      W1a[ky] = half2{l[1], m[1]};
      W1b[ky] = half2{(f16)0.f, r[1]};
    }
    // band rows (from row r0 on).  DOT2: tap pairs of one channel, P0[y][i] = columns (i, i +
    // 1) of k >= 1, Q0[y][j] = columns (j, j + 1) of k = 0, for the pair's first channel, P1
    // and Q1 for its second; else V[y][i] = the channel pair at column i
    half2 P0[G::RPW + 2][TW / 2 + 1], P1[G::RPW + 2][TW / 2 + 1], Q0[G::RPW + 2][2], Q1[G::RPW + 2][2];
    half2 V[G::RPW + 2][TW / 2 + 2];
    half2 out[G::RPW][TW / 2];
    auto band_at = [&](int y, int off) __attribute__((always_inline)) {
      return *(const uint32_t*)(band + y * BROW + ((y & 1) ? off ^ 64 : off));
    };
    // what the outputs k >= 1 and k = 0 of a row need of band row y
    auto load_row = [&](int y, bool rest, bool edge) __attribute__((always_inline)) {
      if constexpr (!DOT2) {
#pragma unroll
        for (int i = 0; i < TW / 2 + 2; ++i) V[y][i] = __builtin_bit_cast(half2, band_at(y, va[i]));
      } else {
        auto lo = [](uint32_t a, uint32_t b) { return __builtin_bit_cast(half2, __builtin_amdgcn_perm(b, a, 0x05040100u)); };
        auto hi = [](uint32_t a, uint32_t b) { return __builtin_bit_cast(half2, __builtin_amdgcn_perm(b, a, 0x07060302u)); };
        uint32_t vr[TW / 2 + 2], er[3];
        if (rest)
#pragma unroll
          for (int i = 1; i < TW / 2 + 2; ++i) vr[i] = band_at(y, va[i]);
        if (edge)
#pragma unroll
          for (int j = 0; j < 3; ++j) er[j] = band_at(y, ve[j]);
        if (rest)
#pragma unroll
          for (int i = 1; i < TW / 2 + 1; ++i) {
            P0[y][i] = lo(vr[i], vr[i + 1]);
            P1[y][i] = hi(vr[i], vr[i + 1]);
          }
        if (edge)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            Q0[y][j] = lo(er[j], er[j + 1]);
            Q1[y][j] = hi(er[j], er[j + 1]);
          }
      }
    };
    // one output (row r, step k) of the channel pair
    auto dw_out = [&](int r, int k) __attribute__((always_inline)) {
      float a0 = bias0, a1 = bias1;
      if constexpr (DOT2) {
#pragma unroll
        for (int y = r; y < r + 3; ++y) {
          a0 = __builtin_amdgcn_fdot2(W0a[y - r], k ? P0[y][k] : Q0[y][0], a0, false);
          a0 = __builtin_amdgcn_fdot2(W0b[y - r], k ? P0[y][k + 1] : Q0[y][1], a0, false);
          a1 = __builtin_amdgcn_fdot2(W1a[y - r], k ? P1[y][k] : Q1[y][0], a1, false);
          a1 = __builtin_amdgcn_fdot2(W1b[y - r], k ? P1[y][k + 1] : Q1[y][1], a1, false);
        }
      } else {
        // even rows, odd columns: the last tap's sum is rounded to fp16 by the fma itself, at
        // the others to fp32 and then to fp16 (fixed here, so that it does not depend on the
        // compiler's choice of instructions; a wait state lies between a half-register result and
        // its reader)
        const bool fused = r % 2 == 0 && k % 2 == 1;
#pragma unroll
        for (int t = 0; t < (fused ? 8 : 9); ++t) {
          const half2 ww = wt[t], zz = V[r + t / 3][k + t % 3];
          a0 = fmaf((float)ww[0], (float)zz[0], a0);
          a1 = fmaf((float)ww[1], (float)zz[1], a1);
        }
        if (fused) {
          asm("v_fma_mixlo_f16 %0, %1, %2, %3 op_sel_hi:[1,1,0]\n\ts_nop 0\n\t"
              "v_fma_mixhi_f16 %0, %1, %2, %4 op_sel:[1,1,0] op_sel_hi:[1,1,0]\n\ts_nop 0"
              : "=&v"(out[r][k])
              : "v"(wt[8]), "v"(V[r + 2][k + 2]), "v"(a0), "v"(a1));
          return;
        }
        asm("" : "+v"(a0), "+v"(a1));
      }
      out[r][k] = half2{(f16)a0, (f16)a1};
    };
    // the residual of the wave's outputs is the band's interior: lane = pixel
    // 32 g + lane % 32, unit 4 (t % 2) + 2 q + lane / 32 of group t / 2
    auto read_res = [&]() __attribute__((always_inline)) {
      const int n = lane & 31, y = n >> 3, x = 1 + (n & 7);
#pragma unroll
      for (int c = 0; c < G::T2; ++c) {
        const int t = tile0 + c;
        const char* rb = smem + (t >> 1) * REG + (1 + y) * BROW + x * 128;
        const int f = (4 * (t & 1) + h) ^ usw(1 + y, x);
#pragma unroll
        for (int g = 0; g < G::G2; ++g)
#pragma unroll
          for (int q = 0; q < 2; ++q)
            res[c][g][q] = *(const half8*)(rb + 4 * (g2 + g) * BROW + ((f ^ (2 * q)) << 4));
      }
    };
    auto dw_rows = [&]() __attribute__((always_inline)) {
      load_row(0, true, true);
      load_row(1, true, true);
#pragma unroll
      for (int r = 0; r < G::RPW; ++r) {
        load_row(r + 2, true, true);
#pragma unroll
        for (int k = 0; k < TW / 2; ++k) dw_out(r, k);
      }
    };
    if constexpr (FIRST) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      if constexpr (!LAST) chain_count_in(run, tile);
      lds_barrier();
      read_res();
      dw_rows();
    } else {
      // before this block's ring is known: the outputs that read only the
      // interior (rows 1 .. 6, columns 1 .. 6), where a wave holds all rows,
      // and the residual
      read_res();
      if constexpr (G::RPW == TH) {
        load_row(1, true, false);
        load_row(2, true, false);
#pragma unroll
        for (int r = 1; r <= TH - 2; ++r) {
          load_row(r + 2, true, false);
#pragma unroll
          for (int k = 1; k < TW / 2; ++k) dw_out(r, k);
        }
      }
      // the ring, once every neighbouring tile has published block b - 1 (its
      // edge pixels are in a.src)
      if (wave == 0) chain_wait(run, b, lane, tyi, txi, tiles_y, tiles_x);
      lds_barrier();
      // the ring (36 pixels: rows -1 and 8, columns -1 and 8 of rows 0 .. 7)
      // through registers, split over the group's waves; device-coherent
      // loads, which bypass this XCD's L2 (it may hold an older copy of the
      // line): the neighbours wrote these pixels in this launch
      constexpr int RING = 2 * BW + 2 * TH;
      constexpr int NR = (RING * 8 / G::RW + 63) / 64;
      static_assert(RING * 8 % G::RW == 0, "ring units per wave");
      half8 rv[NR];
      const f16* rp[NR];
      int ro[NR];
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        const int T = i * 64 + lane;
        const bool mine = T < RING * 8 / G::RW;
        const int S = G::RW == 1 ? T : (wave % G::RW) * (RING * 8 / G::RW) + T;
        const int r = S >> 3, u = S & 7;
        const int by = r < BW ? 0 : r < 2 * BW ? BH - 1 : 1 + ((r - 2 * BW) & (TH - 1));
        const int bx = r < BW ? r : r < 2 * BW ? r - BW : (r < 2 * BW + TH ? 0 : BW - 1);
        const int hy = ty0 - 1 + by, hx = tx0 - 1 + bx;
        const bool in = mine && hy >= 0 && hy < a.h && hx >= 0 && hx < a.w;
        rp[i] = in ? z + (size_t)(hy * a.w + hx) * C + 64 * cg + 8 * u : zpad;
        ro[i] = mine ? by * BROW + bx * 128 + ((u ^ usw(by, bx)) << 4) : -1;
      }
      load_coherent16(rv, rp);
#pragma unroll
      for (int i = 0; i < NR; ++i)
        if (ro[i] >= 0) *(half8*)(band + ro[i]) = rv[i];
      if constexpr (G::RPW == TH) {
        // the outputs that read the ring
        load_row(0, true, true);
        load_row(1, true, true);
        load_row(2, true, true);
#pragma unroll
        for (int k = 0; k < TW / 2; ++k) dw_out(0, k);
#pragma unroll
        for (int r = 1; r <= TH - 2; ++r) {
          load_row(r + 2, r >= TH - 3, true);
          dw_out(r, 0);
        }
        load_row(TH + 1, true, true);
#pragma unroll
        for (int k = 0; k < TW / 2; ++k) dw_out(TH - 1, k);
      } else {
        lds_barrier();  // the group's whole ring is in
        dw_rows();
      }
    }
    // the band has been read (by every wave of its group) before a goes over it
    if constexpr (G::RW > 1) lds_barrier();
    if (bi < 3 * C / 4) *(floatx4*)(smem + G::OBIAS + 16 * bi) = bv;
    // output (row r, step k): column x(k), a's fragment (group r / 4, k-step 4 cg + cp /
    // 8), lane slot 8 (r % 4) + x + 32 kh, kh = (cp / 4) % 2 (bslot of it: side = half, kk
    // = x or 7 - x), elements 2 (cp % 4), + 1
    const int kh = (cp >> 2) & 1;
    int fo[2];
#pragma unroll
    for (int par = 0; par < 2; ++par)
      fo[par] = cg * REG + (cp >> 3) * XF + (cp & 3) * 4 + (32 * kh + 4 * ((half + 2 * par + 2 * kh) & 3)) * 16;
    int kk[TW / 2];
#pragma unroll
    for (int k = 0; k < TW / 2; ++k) kk[k] = 16 * (DOT2 ? (role ? (4 - k) & 3 : k) : (half ? 3 - k : k));
#pragma unroll
    for (int r = 0; r < G::RPW; ++r) {
      const int rr = r0 + r;
#pragma unroll
      for (int k = 0; k < TW / 2; ++k)
        *(half2*)(smem + fo[r & 1] + kk[k] + (rr >> 2) * 4 * XF + ((rr >> 1) & 1) * 256) = out[r][k];
    }
  }
  lds_barrier();  // a and the biases complete; every wave holds its residual
  if constexpr (FIRST && !LAST) chain_tell(run, smem + G::SYNC);

  // ---- 2, 3. pw1 and pw2
  floatx16 acc[2][2];
  auto init_acc = [&](int c, int row, int ng) __attribute__((always_inline)) {
    const float* bp = (const float*)(smem + G::OBIAS) + row + 4 * h;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const floatx4 v = *(const floatx4*)(bp + 8 * q);
#pragma unroll
      for (int g = 0; g < 2; ++g)
        if (g < ng)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[c][g][4 * q + e] = v[e];
    }
  };
  auto init_pw1 = [&](int r) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < G::C1; ++c) {
      const int e = entry(r, c);
      init_acc(c, GATED ? c * C + 32 * (e >> 1) : 32 * e, G::G1);
    }
  };
  // Hand-off of round r: the hidden values as pw2 B fragments (the pw2 weights
  // are packed in the accumulators' register order).  LeakyReLU: C = 64 and 128 in fp32,
  // rounded to fp16 once; C = 256 max(h, 0.1 h) of the fp16-rounded value, in packed fp16.
  // Gated: WSiLU(h1) = h1 sigmoid(4 h1) rounded to fp16, then g = WSiLU(h1) h2 rounded to fp16.
  auto handoff = [&](int r) __attribute__((always_inline)) {
#pragma unroll
    for (int g = 0; g < G::G1; ++g)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if constexpr (GATED) {
          half8 gv;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float h1 = acc[0][g][8 * u + e];
            const f16 ws = (f16)(h1 / (1.f + __expf(-4.f * h1)));
            gv[e] = (f16)((float)ws * acc[1][g][8 * u + e]);
          }
          const int k = 2 * pair0 + u;
          *(half8*)(smem + (r ? G::h1_off(g1 + g, k) : G::h0_off(g1 + g, k)) + myslot) = gv;
        } else {
#pragma unroll
          for (int c = 0; c < G::C1; ++c) {
            half8 gv;
            if constexpr (C < 256) {
#pragma unroll
              for (int e = 0; e < 8; ++e) gv[e] = (f16)leaky(acc[c][g][8 * u + e]);
            } else {
              half8 hv;
#pragma unroll
              for (int e = 0; e < 8; ++e) hv[e] = (f16)acc[c][g][8 * u + e];
              const half8 sl = hv * (f16)0.1f;
#pragma unroll
              for (int e = 0; e < 8; ++e) gv[e] = __builtin_fmaxf16(hv[e], sl[e]);
            }
            const int k = 2 * G::C1 * wave + 2 * c + u;
            *(half8*)(smem + (r ? G::h1_off(g, k) : G::h0_off(g, k)) + myslot) = gv;
          }
        }
      }
  };
  // The residual enters the pw2 sums through the identity (the two 32 x 16 halves as A,
  // exact products), at C = 256 before the hidden layer, at C = 64 and 128 after it.
  auto add_res = [&]() __attribute__((always_inline)) {
    const int row = lane & 31;
    half8 e0, e1;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      e0[e] = (f16)(row == 8 * h + e ? 1.f : 0.f);
      e1[e] = (f16)(row == 16 + 8 * h + e ? 1.f : 0.f);
    }
#pragma unroll
    for (int c = 0; c < G::T2; ++c)
#pragma unroll
      for (int g = 0; g < G::G2; ++g)
#pragma unroll
        for (int q = 0; q < 2; ++q) acc[c][g] = mfma_f16(q ? e1 : e0, res[c][g][q], acc[c][g]);
  };
  auto ngroup = [](int t) constexpr { return t < N1 ? G::G1 : G::G2; };
  // B fragment g of the wave at step t
  auto bfrag = [&](int t, int g) __attribute__((always_inline)) {
    int off;
    if (t < N1) {
      off = G::a_off(g1 + g, t % KS);
    } else {
      const int k = t - N1;
      off = k < KH ? G::h0_off(g2 + g, k) : G::h1_off(g2 + g, k - KH);
    }
    return *(const half8*)(smem + off + myslot);
  };
  half8 qb[PB][2];
  auto start_b = [&](int t) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < PB; ++s)
#pragma unroll
      for (int g = 0; g < 2; ++g)
        if (g < ngroup(t)) qb[(t + s) % PB][g] = bfrag(t + s, g);
  };
  init_pw1(0);
  start_b(0);
  __builtin_amdgcn_sched_barrier(0);
  auto step = [&](auto tc) __attribute__((always_inline)) {
    constexpr int t = decltype(tc)::value;
    if constexpr (G::R == 2 && t == KS) {
      // round 0 done: its hidden fragments go where no one reads before the
      // hand-off barrier, then round 1 from its bias
      handoff(0);
      init_pw1(1);
    }
    if constexpr (t == N1) {
      // the last round: with two rounds its hidden fragments replace a, once
      // every wave is past its last read of a (the MFMAs read their operands
      // at issue)
      if constexpr (G::R == 2) lds_barrier();
      handoff(G::R - 1);
      // the pw2 accumulators start from the bias
#pragma unroll
      for (int c = 0; c < G::T2; ++c) init_acc(c, 2 * C + 32 * (tile0 + c), G::G2);
      if constexpr (C == 256) add_res();
      lds_barrier();
      start_b(t);
    }
    half8 A[2], B[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      if (c < nfrag(t)) A[c] = qa[t % PA][c];
      if (t + PA < NT && c < nfrag(t + PA)) qa[t % PA][c] = afrag(t + PA, c);
    }
    // the B window restarts at the hand-off to pw2
    constexpr bool bnext = t + PB < NT && (t >= N1 || t + PB < N1);
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      if (g < ngroup(t)) B[g] = qb[t % PB][g];
      if (bnext && g < ngroup(t + PB)) qb[t % PB][g] = bfrag(t + PB, g);
    }
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int g = 0; g < 2; ++g)
        if (c < nfrag(t) && g < ngroup(t)) acc[c][g] = mfma_f16(A[c], B[g], acc[c][g]);
    __builtin_amdgcn_sched_barrier(0);
  };
  unrolled(step, std::make_integer_sequence<int, NT>{});
  if constexpr (C < 256) add_res();

  bool late = false;
  if constexpr (FIRST && !LAST) late = chain_too_late(run, smem + G::SYNC);
  lds_barrier();  // every wave is done reading the hidden layer
  // ---- the output, rounded to fp16 once, into the interior of the bands:
  // pixel (1 + y, 1 + x), 16-byte unit 4 (t % 2) + q, half h, of group t / 2;
  // zero outside the image (the next depthwise's padding)
  const bool full = ty0 + TH <= a.h && tx0 + TW <= a.w;
#pragma unroll
  for (int g = 0; g < G::G2; ++g) {
    const int p = 32 * (g2 + g) + (lane & 31), py = p >> 3, px = p & 7;
    const int sw = usw(1 + py, 1 + px);
    const bool zero = !full && !(ty0 + py < a.h && tx0 + px < a.w);
#pragma unroll
    for (int c = 0; c < G::T2; ++c) {
      const int t = tile0 + c;
      char* const pb = smem + (t >> 1) * REG + (1 + py) * BROW + (1 + px) * 128 + 8 * h;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        half4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = zero ? (f16)0.f : (f16)acc[c][g][4 * q + e];
        *(half4*)(pb + (((4 * (t & 1) + q) ^ sw) << 4)) = o;
      }
    }
  }
  lds_barrier();
  f16* dst = (f16*)a.dst;
  if constexpr (LAST) {
    if constexpr (C == 256) {
      if (down && ca->down_w) {
        dc64_down(smem, *ca, a, ty0, tx0, wave, lane);
        return true;
      }
    }
    // whole pixels as 16-byte vectors
    constexpr int U = C / 8;  // units per pixel
#pragma unroll
    for (int i = 0; i < TH * TW * U / 256; ++i) {
      const int idx = i * 256 + threadIdx.x;
      const int p = idx / U, u = idx % U, py = p >> 3, px = p & 7;
      const int yy = ty0 + py, xx = tx0 + px;
      if (yy < a.h && xx < a.w) {
        const half8 v = *(const half8*)(smem + (u >> 3) * REG + (1 + py) * BROW + (1 + px) * 128 +
                                        (((u & 7) ^ usw(1 + py, 1 + px)) << 4));
        __builtin_nontemporal_store(v, (half8*)(dst + (size_t)(yy * a.w + xx) * C + 8 * u));
      }
    }
  } else {
    if (FIRST && late) return false;
    // the tile's 28 edge pixels, from the bands to memory for the neighbours' rings
    constexpr int EDGE = 2 * TW + 2 * (TH - 2);
    constexpr int NE = EDGE * (C / 8);
#pragma unroll
    for (int i = 0; i < (NE + 255) / 256; ++i) {
      const int S = i * 256 + threadIdx.x;
      // 8 consecutive lanes: one pixel's 64 channels of a group
      const int u = S & 7, cgp = (S >> 3) % G::NG, e = (S >> 3) / G::NG;
      // edge e: row 0 (e < 8), row 7 (e < 16), column 0 of rows 1 .. 6 (e < 22), column 7 of rows 1 .. 6
      const int e6 = e - 2 * TW, side = e6 >= TH - 2 ? 1 : 0;
      const int py = e < TW ? 0 : e < 2 * TW ? TH - 1 : 1 + e6 - side * (TH - 2);
      const int px = e < TW ? e : e < 2 * TW ? e - TW : side * (TW - 1);
      const int yy = ty0 + py, xx = tx0 + px;
      if (S < NE && yy < a.h && xx < a.w) {
        const half8 v = *(const half8*)(smem + cgp * REG + (1 + py) * BROW + (1 + px) * 128 +
                                        ((u ^ usw(1 + py, 1 + px)) << 4));
        store_coherent16(dst + (size_t)(yy * a.w + xx) * C + 64 * cgp + 8 * u, v);
      }
    }
    // publish: every wave's edge stores are complete at the device's point of
    // coherence (their acknowledgements counted down) before the tile's word
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();
    chain_publish(run, tile, b);
  }
  return true;
}

// Workgroup -> tile: the first 256 workgroups (one per CU) take the first 256
// tiles, the next 256 the following ones, each range XCD by XCD, so that the
// two tiles that share a CU lie far apart in the frame: in a chain they may
// then run half a block out of step, one in its MFMA loops while the other is
// in its VALU and memory phases.  (Left to themselves the first of the two, the older,
// always goes first; the frame's second half then falls two blocks behind and
// its neighbours wait.  With the lead alternating from block to block a gated 1080p encode
// takes 435 us instead of 451, a decode 196.6 instead of 197.2.)
__device__ __forceinline__ int dc64_tile() {
  const int slot = blockIdx.x >> 8, n = min(256, (int)gridDim.x - (slot << 8));
  return (slot << 8) + xcd_tile(blockIdx.x & 255, n);
}

template <int C, bool GATED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(Geo<C, GATED>::WPE, Geo<C, GATED>::WPE)))
void k_dcblock64_f16(BlockArgs a) {
  __shared__ __attribute__((aligned(1024))) char smem[Geo<C, GATED>::SMEM];
  const int tiles_x = (a.w + TW - 1) / TW, tiles_y = (a.h + TH - 1) / TH;
  const int tile = dc64_tile();
  if (tile >= tiles_x * tiles_y) return;
  const int wave0 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  ChainRun none{};
  dc64_block<C, GATED, true, true>(smem, a, 0, tile, tiles_x, tiles_y, wave0, none, nullptr, false);
}

// A chain: blocks 0 .. nb - 1 of a transform in one launch (blk[b] reads
// blk[b - 1].dst).  Each tile keeps its block output in LDS, in the interior
// of the next block's band, so between blocks only the ring of the band (the
// neighbours' edge pixels) moves through memory: a block other than the last
// stores only the tile's 28 edge pixels, then publishes its progress in
// its word; the next block waits until every neighbouring tile has published
// that block, then reads its ring.  The host launches a chain where the device holds
// every tile of the grid at once; a launch that finds itself without room for them
// all runs block by block with those that are there (chain_sync.hpp).
template <int C, bool GATED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(Geo<C, GATED>::WPE, Geo<C, GATED>::WPE)))
void k_dcchain64_f16(DcChainArgs ca) {
  __shared__ __attribute__((aligned(1024))) char smem[Geo<C, GATED>::SMEM];
  const int tiles_x = (ca.blk[0].w + TW - 1) / TW, tiles_y = (ca.blk[0].h + TH - 1) / TH;
  const int tile = dc64_tile();
  if (tile >= tiles_x * tiles_y) return;
  const int wave0 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nb = ca.nb;
  ChainRun run = chain_begin(ca, tile, tiles_x * tiles_y);
  if (!dc64_block<C, GATED, true, false>(smem, ca.blk[0], 0, tile, tiles_x, tiles_y, wave0, run, &ca)) {
    chain_end(run, tile);
    return;
  }
  if (!chain_goes_on(run)) {
    chain_sealed(run, nb, (uint32_t*)(smem + Geo<C, GATED>::SYNC), [&](int b, int t) __attribute__((always_inline)) {
      dc64_block<C, GATED, true, true>(smem, ca.blk[b], 0, t, tiles_x, tiles_y, wave0, run, &ca, b == nb - 1);
    });
    chain_end(run, tile);
    return;
  }
  for (int i = 1; i < nb - 1; ++i) {
    const int b = __builtin_amdgcn_readfirstlane(i);  // uniform for the compiler too: scalar loads of the arguments
    dc64_block<C, GATED, false, false>(smem, ca.blk[b], b, tile, tiles_x, tiles_y, wave0, run, &ca);
  }
  dc64_block<C, GATED, false, true>(smem, ca.blk[nb - 1], nb - 1, tile, tiles_x, tiles_y, wave0, run, &ca);
}

template <int C>
hipError_t launch_block(bool gated, const BlockArgs& a, hipStream_t st) {
  const dim3 grid(dc64_grid(a.h, a.w));
  if (gated) launch(k_dcblock64_f16<C, true>, grid, dim3(256), st, a);
  else launch(k_dcblock64_f16<C, false>, grid, dim3(256), st, a);
  return hipGetLastError();
}

template <int C>
hipError_t launch_chain(bool gated, const DcChainArgs& ca, hipStream_t st) {
  const dim3 grid(dc64_grid(ca.blk[0].h, ca.blk[0].w));
  if (gated) launch(k_dcchain64_f16<C, true>, grid, dim3(256), st, ca);
  else launch(k_dcchain64_f16<C, false>, grid, dim3(256), st, ca);
  return hipGetLastError();
}

template <int C>
int resident(bool gated) {
  int dev = 0, per_cu = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  const hipError_t e = gated ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_dcchain64_f16<C, true>, 256, 0)
                             : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_dcchain64_f16<C, false>, 256, 0);
  return e == hipSuccess ? per_cu * cus : 0;
}

}  // namespace

hipError_t launch_dcblock64_f16(int C, bool gated, const BlockArgs& a, hipStream_t st) {
  switch (C) {
    case 64: return launch_block<64>(gated, a, st);
    case 128: return launch_block<128>(gated, a, st);
    case 256: return launch_block<256>(gated, a, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_dcchain64_f16(int C, bool gated, const DcChainArgs& ca, hipStream_t st) {
  if (ca.nb < 2 || ca.nb > kMaxChain) return hipErrorInvalidValue;
  switch (C) {
    case 64: return launch_chain<64>(gated, ca, st);
    case 128: return launch_chain<128>(gated, ca, st);
    case 256: return launch_chain<256>(gated, ca, st);
  }
  return hipErrorInvalidValue;
}

int dcchain64_resident(int C, bool gated) {
  switch (C) {
    case 64: return resident<64>(gated);
    case 128: return resident<128>(gated);
    case 256: return resident<256>(gated);
  }
  return 0;
}

}  // namespace nc
