// int16 DC block (Sec. 4.5, Alg. 1; LeakyReLU and gated forms), C = 64, 128 and 256, on
// 8 x 8 pixel tiles, one block per launch or a chain of blocks: the fp16 kernel's
// tiles, waves, LDS layout and exchange (kernels_f16_dc64.hip) with integer arithmetic.
//   - An int16 x int16 product is four int8 digit products (x = 256 xh + xl' + 128, w =
//     256 wh + wl).  Two accumulators per tile and pixel group, both fed by one pass over
//     the high weight digits (H += wh xh, L += wh xl), then H = 256 H + L and one
//     pass over the low ones, L from the correction: 256 H + L = 65536 hh + 256 (hl + lh) + ll + corr in
//     wrapping int32.  Each weight fragment feeds four MFMAs and is read once.
//   - Depthwise: v_dot2_i32_i16, rescaled, the two lanes of a channel quad swapping
//     their pairs through DPP; one keeps the quad's high digits, the other its low digits.
//   - Hand-offs rescale, apply the integer LeakyReLU or the gate (sigmoid table in LDS)
//     and split into digits; the output adds the residual with saturation.
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
constexpr int kSigSat = 888;   // S[v] = 512 from here on
constexpr int kSigBytes = 896; // the compact sigmoid table, padded to 16-byte units
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
  static constexpr int KS = C / 32;                 // pw1 k-steps of a pass
  static constexpr int MT = C / 32;                 // pw2 output tiles
  static constexpr int FR = 2 * KS + 2 * MT;        // fragments per hidden chunk in the weight image
  static constexpr int NG = C / 64;                 // channel groups
  static constexpr int RW = 4 / NG;                 // waves that share a channel group
  static constexpr int RPW = TH / RW;               // output rows per wave
  static constexpr int R = C == 256 ? 2 : 1;        // pw1 rounds
  static constexpr int C1 = C == 64 && !GATED ? 1 : 2;  // pw1 chunks per wave and round
  static constexpr int G1 = C == 64 && GATED ? 1 : 2;   // pixel groups of a wave's pw1
  static constexpr int T2 = C == 256 ? 2 : 1;       // pw2 output tiles per wave
  static constexpr int G2 = C == 64 ? 1 : 2;        // pixel groups of a wave's pw2
  static constexpr int K2 = (GATED ? C : 2 * C) / 32;  // pw2 k-steps of a pass
  static constexpr int KH = K2 / R;                 // of them per round
  static constexpr int N1 = R * 2 * KS;             // weight-stream steps of pw1 (two passes a round)
  static constexpr int NT = N1 + 2 * K2;
  static constexpr int HF = 2 * KH;                 // hidden fragments (k-step, digit) per round and group
  // LDS: the regions, fragments of the hidden layer that do not fit there, biases
  static constexpr int OX = NG * REG;
  static constexpr int NX = C == 256 ? (GATED ? 0 : 16) : 2 * HF;
  static constexpr int OBIAS = OX + NX * XF;
  static constexpr int OSIG = OBIAS + 12 * C;
  static constexpr int SMEM = OSIG + (GATED ? kSigBytes : 0);
  static constexpr int SYNC = REG - 16;  // a word no one else uses once the first band is in
  // registers per lane allow 2 workgroups per CU
  static constexpr int WPE = 2;
  static_assert(SMEM * WPE <= 160 * 1024, "WPE workgroups fit the LDS of a CU");

  // a's fragment (pixel group g, s = 2 k-step + digit)
  static __device__ __forceinline__ constexpr int a_off(int g, int s) {
    return (s >> 2) * REG + (4 * g + (s & 3)) * XF;
  }
  // hidden fragment (g, k = 2 k-step + digit) of round 0
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

typedef short short2v __attribute__((ext_vector_type(2)));

// RHE(a / 8192) for any int32 a, before the saturation to int16 (|a| >= 2^28
// saturates either way, so a is clamped first; then the round-half-even bias
// add stays in range).
__device__ __forceinline__ int rhe13(int a) {
  const int ac = min(max(a, -(1 << 28)), 1 << 28);
  return (ac + 4095 + ((ac >> 13) & 1)) >> 13;
}
// clip(RHE(a / 8192)) to int16 for any int32 a: clamping a to
// [-2^28, 2^28 - 4097] first gives the saturated value directly.
__device__ __forceinline__ int rescale13c(int a) {
  const int ac = min(max(a, -(1 << 28)), (1 << 28) - 4097);
  return (ac + 4095 + ((ac >> 13) & 1)) >> 13;
}
// RHE(m / 512) for |m| <= 2^30
__device__ __forceinline__ int rhe9(int m) { return (m + 255 + ((m >> 9) & 1)) >> 9; }
// S[v] from the compact table: 512 from |v| = 888 on, S[-v] = 512 - S[v]
__device__ __forceinline__ int sigmoid_of(int v, const uint8_t* s8) {
  const int a = v < 0 ? -v : v;
  const int sa = a >= kSigSat ? 512 : 256 + (int)s8[min(a, kSigSat - 1)];  // index kept in the table
  return v < 0 ? 512 - sa : sa;
}
// Two int32 values saturated to int16 and packed (first in the low half).
__device__ __forceinline__ uint32_t pack_sat(int lo, int hi) {
  return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pk_i16(lo, hi));
}
// High digits (signed) and low digits offset by -128 of the four int16 values
// of dwords d0 (first two) and d1 (last two).
__device__ __forceinline__ uint32_t digits_hi(uint32_t d0, uint32_t d1) {
  return __builtin_amdgcn_perm(d1, d0, 0x07050301u);
}
__device__ __forceinline__ uint32_t digits_lo(uint32_t d0, uint32_t d1) {
  return __builtin_amdgcn_perm(d1, d0, 0x06040200u) ^ 0x80808080u;
}

// One block of a tile (FIRST: its band comes whole from a.src; LAST: its
// output goes whole to a.dst; otherwise the chain's ring and edge exchange).
template <int C, bool GATED, bool FIRST, bool LAST>
__device__ __forceinline__ bool dci64_block(char* smem, const BlockArgs& a, int b, int tile, int tiles_x, int tiles_y,
                                           int wave0, ChainRun& run) {
  using G = Geo<C, GATED>;
  constexpr int KS = G::KS, FR = G::FR, NT = G::NT, N1 = G::N1, K2 = G::K2, MT = G::MT;
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
  const int16_t* z = (const int16_t*)a.src;
  const int16_t* zpad = (const int16_t*)a.zpad;
  const char* w1 = (const char*)a.w1;
  // entry (hidden chunk) of the wave's chain c in round r, its pw2 tile t, its pixel groups
  const int pair0 = C == 64 ? wave >> 1 : wave;
  auto entry = [&](int r, int c) __attribute__((always_inline)) {
    if (GATED) return 2 * (4 * r + pair0) + c;
    return C == 64 ? wave : 8 * r + 2 * wave + c;
  };
  const int tile0 = C == 256 ? 2 * wave : C == 128 ? wave : wave >> 1;
  const int g1 = G::G1 == 1 ? wave & 1 : 0, g2 = G::G2 == 1 ? wave & 1 : 0;
  // fragment c of weight-stream step t: pw1 round t / (2 KS), its pass (t / KS) % 2 (the
  // weight digit), then pw2 pass (t - N1) / K2 over the hidden chunks
  auto afrag = [&](int t, int c) __attribute__((always_inline)) {
    int f;
    if (t < N1) {
      f = entry(t / (2 * KS), c) * FR + t % (2 * KS);
    } else {
      const int p = (t - N1) / K2, k = (t - N1) % K2;
      f = (GATED ? 2 * k + 1 : k) * FR + 2 * KS + p * MT + tile0 + c;
    }
    return *(const intx4*)(w1 + (size_t)f * 1024 + lane16);
  };
  // of the two tiles on a CU, one leads in even blocks, the other in odd ones
  if constexpr (!(FIRST && LAST)) {
    if ((b ^ (blockIdx.x >> 8)) & 1) __builtin_amdgcn_s_setprio(1);
    else __builtin_amdgcn_s_setprio(0);
  }
  constexpr int PA = 3, PB = 1;  // prefetch distances (steps) of the A and B windows
  intx4 qa[PA][2];
  auto nfrag = [](int t) constexpr { return t < N1 ? G::C1 : G::T2; };

  // ---- 1. depthwise: channel group cg, rows r0 .. r0 + RPW - 1
  intx2 res[G::T2][G::G2][4];  // residual: (output tile, group, register quad q), 4 int16
  {
    const int cg = G::RW == 1 ? wave : wave / G::RW;
    const int r0 = G::RW == 1 ? 0 : (wave % G::RW) * G::RPW;
    const int cp = lane & 31, half = lane >> 5;
    const int odd = cp & 1;
    // taps of the lane's channel pair as int16 pairs and its two biases 512 b, from
    // the 96-byte record of its channel quad
    uint32_t wt[9];
    int bias0, bias1;
    {
      const intx4* wsrc = (const intx4*)a.dww + 6 * (16 * cg + (cp >> 1));
      intx4 q0 = wsrc[0], q1 = wsrc[1], q2 = wsrc[2], q3 = wsrc[3], q4 = wsrc[4];
      intx2 q5 = *(const intx2*)(wsrc + 5);
      asm volatile("" : "+v"(q0), "+v"(q1), "+v"(q2), "+v"(q3), "+v"(q4), "+v"(q5));
      int wd[22];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        wd[i] = q0[i];
        wd[4 + i] = q1[i];
        wd[8 + i] = q2[i];
        wd[12 + i] = q3[i];
        wd[16 + i] = q4[i];
      }
      wd[20] = q5[0];
      wd[21] = q5[1];
      // wd[i] for the even lane, wd[j] for the odd one, selected by mask (a
      // conditional index would put wd in scratch memory)
      const uint32_t msk = 0u - (uint32_t)odd;
      auto sel = [&](int i, int j) __attribute__((always_inline)) {
        return (uint32_t)wd[i] ^ (((uint32_t)wd[i] ^ (uint32_t)wd[j]) & msk);
      };
#pragma unroll
      for (int t = 0; t < 9; ++t) wt[t] = sel(2 * t, 2 * t + 1);  // tap t: pair 0 or 1 of the quad
      bias0 = (int)sel(18, 20);  // biases of the quad's channels 0 .. 3 at words 18 .. 21
      bias1 = (int)sel(19, 21);
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
    // the block's corrections (pw1 2C, pw2 C, int32), then the sigmoid table, through registers
    intx4 bv = {};
    const int bi = wave * 64 + lane;
    constexpr int NB = 3 * C / 4 + (GATED ? kSigBytes / 16 : 0);
    static_assert(NB <= 256, "one unit per thread");
    if (bi < NB)
      bv = bi < C / 2       ? ((const intx4*)a.b1)[bi]
           : bi < 3 * C / 4 ? ((const intx4*)a.b2)[bi - C / 2]
                            : ((const intx4*)a.sig8)[bi - 3 * C / 4];
    // the first weight fragments
#pragma unroll
    for (int s = 0; s < PA; ++s)
#pragma unroll
      for (int c = 0; c < 2; ++c)
        if (c < nfrag(s)) qa[s][c] = afrag(s, c);
    // the lane's band reads: column i (half 0) or 9 - i (half 1) of a row, its
    // channel pair's dword; rows of odd index at va ^ 64
    int va[TW / 2 + 2];
#pragma unroll
    for (int i = 0; i < TW / 2 + 2; ++i) {
      const int col = half ? TW + 1 - i : i;
      va[i] = r0 * BROW + col * 128 + (((cp >> 2) ^ usw(0, col)) << 4) + (cp & 3) * 4;
    }
    // taps of a row as dot2 pairs (mirrored for half 1): (A0, A1) . (z[k],
    // z[k + 1]) and (0, A2) . (z[k + 1], z[k + 2]) in the lane's column order
    uint32_t W0a[3], W0b[3], W1a[3], W1b[3];
#pragma unroll
    for (int ky = 0; ky < 3; ++ky) {
      const uint32_t l = half ? wt[3 * ky + 2] : wt[3 * ky], m = wt[3 * ky + 1], r = half ? wt[3 * ky] : wt[3 * ky + 2];
      W0a[ky] = __builtin_amdgcn_perm(m, l, 0x05040100u);
      W0b[ky] = r << 16;
      W1a[ky] = __builtin_amdgcn_perm(m, l, 0x07060302u);
      W1b[ky] = r & 0xFFFF0000u;
    }
    // band rows (from row r0 on) as tap pairs of one channel: P0[y][i] =
    // (z[y][i], z[y][i + 1]) of the pair's first channel, P1 of its second
    uint32_t P0[G::RPW + 2][TW / 2 + 1], P1[G::RPW + 2][TW / 2 + 1];
    uint32_t out[G::RPW][TW / 2];
    auto load_row = [&](int y, int i0) __attribute__((always_inline)) {
      uint32_t vr[TW / 2 + 2];
#pragma unroll
      for (int i = 0; i < TW / 2 + 2; ++i)
        if (i >= i0) vr[i] = *(const uint32_t*)(band + y * BROW + ((y & 1) ? va[i] ^ 64 : va[i]));
#pragma unroll
      for (int i = 0; i < TW / 2 + 1; ++i)
        if (i >= i0) {
          P0[y][i] = __builtin_amdgcn_perm(vr[i + 1], vr[i], 0x05040100u);
          P1[y][i] = __builtin_amdgcn_perm(vr[i + 1], vr[i], 0x07060302u);
        }
    };
    // one output (row r, step k) of the channel pair; the even lane of a quad keeps
    // the high digits of (own pair, partner's), the odd lane the low digits of
    // (partner's, own)
    const uint32_t dsel = odd ? 0x02000604u : 0x07050301u, dxor = odd ? 0x80808080u : 0u;
    auto sdot = [](uint32_t w, uint32_t v, int acc) __attribute__((always_inline)) {
      return __builtin_amdgcn_sdot2(__builtin_bit_cast(short2v, w), __builtin_bit_cast(short2v, v), acc, false);
    };
    auto dw_out = [&](int r, int k) __attribute__((always_inline)) {
      int a0 = bias0, a1 = bias1;
#pragma unroll
      for (int ky = 0; ky < 3; ++ky) {
        a0 = sdot(W0a[ky], P0[r + ky][k], a0);
        a0 = sdot(W0b[ky], P0[r + ky][k + 1], a0);
        a1 = sdot(W1a[ky], P1[r + ky][k], a1);
        a1 = sdot(W1b[ky], P1[r + ky][k + 1], a1);
      }
      const uint32_t d = pack_sat(rhe13(a0), rhe13(a1));
      const uint32_t p = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)d, 0xB1, 0xF, 0xF, false);  // lane ^ 1
      out[r][k] = __builtin_amdgcn_perm(p, d, dsel) ^ dxor;
    };
    // the residual of the wave's outputs is the band's interior: lane = pixel 32 g +
    // lane % 32, channels 8 q + 4 h .. + 3 of the tile (unit 4 (t % 2) + q of group t / 2)
    auto read_res = [&]() __attribute__((always_inline)) {
      const int n = lane & 31, y = n >> 3, x = 1 + (n & 7);
#pragma unroll
      for (int c = 0; c < G::T2; ++c) {
        const int t = tile0 + c;
        const char* rb = smem + (t >> 1) * REG + (1 + y) * BROW + x * 128 + 8 * h;
        const int f = (4 * (t & 1)) ^ usw(1 + y, x);
#pragma unroll
        for (int g = 0; g < G::G2; ++g)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            res[c][g][q] = *(const intx2*)(rb + 4 * (g2 + g) * BROW + ((f ^ q) << 4));
      }
    };
    auto dw_rows = [&]() __attribute__((always_inline)) {
      load_row(0, 0);
      load_row(1, 0);
#pragma unroll
      for (int r = 0; r < G::RPW; ++r) {
        load_row(r + 2, 0);
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
        load_row(1, 1);
        load_row(2, 1);
#pragma unroll
        for (int r = 1; r <= TH - 2; ++r) {
          load_row(r + 2, 1);
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
      intx4 rv[NR];
      const int16_t* rp[NR];
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
        if (ro[i] >= 0) *(intx4*)(band + ro[i]) = rv[i];
      if constexpr (G::RPW == TH) {
        // the outputs that read the ring
        load_row(0, 0);
        load_row(1, 0);
        load_row(2, 0);
#pragma unroll
        for (int k = 0; k < TW / 2; ++k) dw_out(0, k);
#pragma unroll
        for (int r = 1; r <= TH - 2; ++r) {
          load_row(r + 2, 0);
          dw_out(r, 0);
        }
        load_row(TH + 1, 0);
#pragma unroll
        for (int k = 0; k < TW / 2; ++k) dw_out(TH - 1, k);
      } else {
        lds_barrier();  // the group's whole ring is in
        dw_rows();
      }
    }
    // the band has been read (by every wave of its group) before a goes over it
    if constexpr (G::RW > 1) lds_barrier();
    if (bi < NB) *(intx4*)(smem + G::OBIAS + 16 * bi) = bv;
    // output (row r, step k): column x = k (half 0) or 7 - k (half 1); its quad's
    // digits go to a's fragments (group r / 4, k-step 2 cg + cp / 16, digit: hi from
    // the even lane, lo from the odd one), lane slot 8 (r % 4) + x + 32 kh, kh = (cp /
    // 8) % 2 (bslot of it: kk = k, side = half), dword (cp / 2) % 4
    const int kh = (cp >> 3) & 1;
    int fo[2];
#pragma unroll
    for (int par = 0; par < 2; ++par)
      fo[par] = cg * REG + (2 * (cp >> 4) + odd) * XF + ((cp >> 1) & 3) * 4 +
                (32 * kh + 4 * ((half + 2 * par + 2 * kh) & 3)) * 16;
#pragma unroll
    for (int r = 0; r < G::RPW; ++r) {
      const int rr = r0 + r;
#pragma unroll
      for (int k = 0; k < TW / 2; ++k)
        *(uint32_t*)(smem + fo[r & 1] + (rr >> 2) * 4 * XF + ((rr >> 1) & 1) * 256 + 16 * k) = out[r][k];
    }
  }
  lds_barrier();  // a and the corrections complete; every wave holds its residual
  if constexpr (FIRST && !LAST) chain_tell(run, smem + G::SYNC);

  // ---- 2, 3. pw1 and pw2
  intx16 accH[2][2], accL[2][2];
  auto zero_acc = [&](int nc, int ng) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int g = 0; g < 2; ++g)
        if (c < nc && g < ng) {
          accH[c][g] = intx16{};
          accL[c][g] = intx16{};
        }
  };
  // between the passes over the high and the low weight digits: H = 256 H + L, L = the
  // correction of rows row(c) + drow(i, h), from LDS
  auto fold_acc = [&](int nc, int ng, auto row) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < 2; ++c)
      if (c < nc) {
        const char* const cp = smem + G::OBIAS + 4 * (row(c) + 4 * h);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const intx4 cv = *(const intx4*)(cp + 32 * q);
#pragma unroll
          for (int g = 0; g < 2; ++g)
            if (g < ng)
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const int i = 4 * q + e;
                accH[c][g][i] = (int)(((uint32_t)accH[c][g][i] << 8) + (uint32_t)accL[c][g][i]);
                accL[c][g][i] = cv[e];
              }
        }
      }
  };
  // the sums of register quad q: 256 H + L
  auto sums = [&](int c, int g, int q) __attribute__((always_inline)) {
    intx4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = (int)(((uint32_t)accH[c][g][4 * q + e] << 8) + (uint32_t)accL[c][g][4 * q + e]);
    return v;
  };
  // Hand-off of round r: rescale, integer LeakyReLU (slope 819 / 8192) as max(h, RHE(819
  // h / 2^13)) or the gate clip(RHE(RHE(h1 S[h1] / 512) h2 / 512)), digits as pw2 B
  // fragments (the pw2 weights are packed in the accumulators' register order)
  auto handoff = [&](int r) __attribute__((always_inline)) {
    const uint8_t* const s8 = (const uint8_t*)(smem + G::OSIG);
#pragma unroll
    for (int c = 0; c < (GATED ? 1 : G::C1); ++c)
#pragma unroll
      for (int g = 0; g < G::G1; ++g) {
        uint32_t d[8];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          int v[4];
          if constexpr (GATED) {
            const intx4 s1 = sums(0, g, q), s2 = sums(1, g, q);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int h1 = rescale13c(s1[e]);
              v[e] = rhe9(rhe9(h1 * sigmoid_of(h1, s8)) * rescale13c(s2[e]));  // |h1 S| <= 2^24, |product| <= 2^30
            }
          } else {
            const intx4 s1 = sums(c, g, q);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int hv = rescale13c(s1[e]);
              const int m = 819 * hv;  // |m| < 2^25
              v[e] = max(hv, (m + 4095 + ((m >> 13) & 1)) >> 13);
            }
          }
          d[2 * q] = pack_sat(v[0], v[1]);
          d[2 * q + 1] = pack_sat(v[2], v[3]);
        }
        intx4 gh, gl;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          gh[i] = (int)digits_hi(d[2 * i], d[2 * i + 1]);
          gl[i] = (int)digits_lo(d[2 * i], d[2 * i + 1]);
        }
        const int f = 2 * (GATED ? pair0 : G::C1 * wave + c);
        *(intx4*)(smem + (r ? G::h1_off(g1 + g, f) : G::h0_off(g1 + g, f)) + myslot) = gh;
        *(intx4*)(smem + (r ? G::h1_off(g1 + g, f + 1) : G::h0_off(g1 + g, f + 1)) + myslot) = gl;
      }
  };
  auto ngroup = [](int t) constexpr { return t < N1 ? G::G1 : G::G2; };
  // B fragment of the wave's group g, digit d at step t
  auto bfrag = [&](int t, int g, int d) __attribute__((always_inline)) {
    int off;
    if (t < N1) {
      off = G::a_off(g1 + g, 2 * (t % KS) + d);
    } else {
      const int k = (t - N1) % K2;
      off = k < G::KH ? G::h0_off(g2 + g, 2 * k + d) : G::h1_off(g2 + g, 2 * (k - G::KH) + d);
    }
    return *(const intx4*)(smem + off + myslot);
  };
  intx4 qb[PB][2][2];
  auto start_b = [&](int t) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < PB; ++s)
#pragma unroll
      for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int d = 0; d < 2; ++d)
          if (g < ngroup(t)) qb[(t + s) % PB][g][d] = bfrag(t + s, g, d);
  };
  zero_acc(G::C1, G::G1);
  start_b(0);
  __builtin_amdgcn_sched_barrier(0);
  auto step = [&](auto tc) __attribute__((always_inline)) {
    constexpr int t = decltype(tc)::value;
    if constexpr (G::R == 2 && t == 2 * KS) {
      // round 0 done: its hidden fragments go where no one reads before the
      // hand-off barrier
      handoff(0);
      zero_acc(G::C1, G::G1);
    }
    if constexpr (t == N1) {
      // the last round: with two rounds its hidden fragments replace a, once
      // every wave is past its last read of a (the MFMAs read their operands
      // at issue)
      if constexpr (G::R == 2) lds_barrier();
      handoff(G::R - 1);
      zero_acc(G::T2, G::G2);
      lds_barrier();
      start_b(t);
    }
    if constexpr (t < N1 && t % (2 * KS) == KS) fold_acc(G::C1, G::G1, [&](int c) { return 32 * entry(t / (2 * KS), c); });
    if constexpr (t == N1 + K2) fold_acc(G::T2, G::G2, [&](int c) { return 2 * C + 32 * (tile0 + c); });
    intx4 A[2], B[2][2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      if (c < nfrag(t)) A[c] = qa[t % PA][c];
      if (t + PA < NT && c < nfrag(t + PA)) qa[t % PA][c] = afrag(t + PA, c);
    }
    // the B window restarts at the hand-off to pw2
    constexpr bool bnext = t + PB < NT && (t >= N1 || t + PB < N1);
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int d = 0; d < 2; ++d) {
        if (g < ngroup(t)) B[g][d] = qb[t % PB][g][d];
        if (bnext && g < ngroup(t + PB)) qb[t % PB][g][d] = bfrag(t + PB, g, d);
      }
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int g = 0; g < 2; ++g)
        if (c < nfrag(t) && g < ngroup(t)) {
          accH[c][g] = mfma_i8(A[c], B[g][0], accH[c][g]);
          accL[c][g] = mfma_i8(A[c], B[g][1], accL[c][g]);
        }
    __builtin_amdgcn_sched_barrier(0);
  };
  unrolled(step, std::make_integer_sequence<int, NT>{});

  bool late = false;
  if constexpr (FIRST && !LAST) late = chain_too_late(run, smem + G::SYNC);
  lds_barrier();  // every wave is done reading the hidden layer
  // ---- the output, clip(residual + clip(RHE(sum / 8192))), into the interior of the
  // bands: pixel (1 + y, 1 + x), 16-byte unit 4 (t % 2) + q, half h, of group t / 2;
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
        const intx4 s4 = sums(c, g, q);
        intx2 o;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          // saturating packed int16 add of the residual pair and the rescaled pair
          // (from inline asm: the vector saturating-add builtin was miscompiled)
          const uint32_t v = pack_sat(rhe13(s4[2 * e]), rhe13(s4[2 * e + 1]));
          const int r = res[c][g][q][e];
          int sum;
          asm("v_pk_add_i16 %0, %1, %2 clamp" : "=v"(sum) : "v"(r), "v"(v));
          o[e] = zero ? 0 : sum;
        }
        *(intx2*)(pb + (((4 * (t & 1) + q) ^ sw) << 4)) = o;
      }
    }
  }
  lds_barrier();
  int16_t* dst = (int16_t*)a.dst;
  if constexpr (LAST) {
    // whole pixels as 16-byte vectors
    constexpr int U = C / 8;  // units per pixel
#pragma unroll
    for (int i = 0; i < TH * TW * U / 256; ++i) {
      const int idx = i * 256 + threadIdx.x;
      const int p = idx / U, u = idx % U, py = p >> 3, px = p & 7;
      const int yy = ty0 + py, xx = tx0 + px;
      if (yy < a.h && xx < a.w) {
        const intx4 v = *(const intx4*)(smem + (u >> 3) * REG + (1 + py) * BROW + (1 + px) * 128 +
                                        (((u & 7) ^ usw(1 + py, 1 + px)) << 4));
        __builtin_nontemporal_store(v, (intx4*)(dst + (size_t)(yy * a.w + xx) * C + 8 * u));
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
        const intx4 v = *(const intx4*)(smem + cgp * REG + (1 + py) * BROW + (1 + px) * 128 +
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
// its neighbours wait.  With the lead alternating from block to block a 1080p decode takes
// 350 us instead of 366, gated 315 instead of 321.)
__device__ __forceinline__ int dci64_tile() {
  const int slot = blockIdx.x >> 8, n = min(256, (int)gridDim.x - (slot << 8));
  return (slot << 8) + xcd_tile(blockIdx.x & 255, n);
}

template <int C, bool GATED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(Geo<C, GATED>::WPE, Geo<C, GATED>::WPE)))
void k_dcblock64_i16(BlockArgs a) {
  __shared__ __attribute__((aligned(1024))) char smem[Geo<C, GATED>::SMEM];
  const int tiles_x = (a.w + TW - 1) / TW, tiles_y = (a.h + TH - 1) / TH;
  const int tile = dci64_tile();
  if (tile >= tiles_x * tiles_y) return;
  const int wave0 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  ChainRun none{};
  dci64_block<C, GATED, true, true>(smem, a, 0, tile, tiles_x, tiles_y, wave0, none);
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
void k_dcchain64_i16(DcChainArgs ca) {
  __shared__ __attribute__((aligned(1024))) char smem[Geo<C, GATED>::SMEM];
  const int tiles_x = (ca.blk[0].w + TW - 1) / TW, tiles_y = (ca.blk[0].h + TH - 1) / TH;
  const int tile = dci64_tile();
  if (tile >= tiles_x * tiles_y) return;
  const int wave0 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nb = ca.nb;
  ChainRun run = chain_begin(ca, tile, tiles_x * tiles_y);
  if (!dci64_block<C, GATED, true, false>(smem, ca.blk[0], 0, tile, tiles_x, tiles_y, wave0, run)) {
    chain_end(run, tile);
    return;
  }
  if (!chain_goes_on(run)) {
    chain_sealed(run, nb, (uint32_t*)(smem + Geo<C, GATED>::SYNC), [&](int b, int t) __attribute__((always_inline)) {
      dci64_block<C, GATED, true, true>(smem, ca.blk[b], 0, t, tiles_x, tiles_y, wave0, run);
    });
    chain_end(run, tile);
    return;
  }
  for (int i = 1; i < nb - 1; ++i) {
    const int b = __builtin_amdgcn_readfirstlane(i);  // uniform for the compiler too: scalar loads of the arguments
    dci64_block<C, GATED, false, false>(smem, ca.blk[b], b, tile, tiles_x, tiles_y, wave0, run);
  }
  dci64_block<C, GATED, false, true>(smem, ca.blk[nb - 1], nb - 1, tile, tiles_x, tiles_y, wave0, run);
}

template <int C>
hipError_t launch_block(bool gated, const BlockArgs& a, hipStream_t st) {
  const dim3 grid(dc64_grid(a.h, a.w));
  if (gated) launch(k_dcblock64_i16<C, true>, grid, dim3(256), st, a);
  else launch(k_dcblock64_i16<C, false>, grid, dim3(256), st, a);
  return hipGetLastError();
}

template <int C>
hipError_t launch_chain(bool gated, const DcChainArgs& ca, hipStream_t st) {
  const dim3 grid(dc64_grid(ca.blk[0].h, ca.blk[0].w));
  if (gated) launch(k_dcchain64_i16<C, true>, grid, dim3(256), st, ca);
  else launch(k_dcchain64_i16<C, false>, grid, dim3(256), st, ca);
  return hipGetLastError();
}

template <int C>
int resident(bool gated) {
  int dev = 0, per_cu = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  const hipError_t e = gated ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_dcchain64_i16<C, true>, 256, 0)
                             : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_dcchain64_i16<C, false>, 256, 0);
  return e == hipSuccess ? per_cu * cus : 0;
}

}  // namespace

hipError_t launch_dcblock64_i16(int C, bool gated, const BlockArgs& a, hipStream_t st) {
  switch (C) {
    case 64: return launch_block<64>(gated, a, st);
    case 128: return launch_block<128>(gated, a, st);
    case 256: return launch_block<256>(gated, a, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_dcchain64_i16(int C, bool gated, const DcChainArgs& ca, hipStream_t st) {
  if (ca.nb < 2 || ca.nb > kMaxChain) return hipErrorInvalidValue;
  switch (C) {
    case 64: return launch_chain<64>(gated, ca, st);
    case 128: return launch_chain<128>(gated, ca, st);
    case 256: return launch_chain<256>(gated, ca, st);
  }
  return hipErrorInvalidValue;
}

int dcchain64_i16_resident(int C, bool gated) {
  switch (C) {
    case 64: return resident<64>(gated);
    case 128: return resident<128>(gated);
    case 256: return resident<256>(gated);
  }
  return 0;
}

}  // namespace nc
