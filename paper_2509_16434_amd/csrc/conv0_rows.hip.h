// The first convolution (one or three input channels, 32 output channels, 3x3 stride 2 pad 1, bias, ReLU) produced row by row
// in LDS for the second layer's kernels, so that its output - the largest tensor of the network, 8 times the image of one
// channel, 8/3 times that of three - is neither written nor read back.
//
// A wave makes 32 pixels x 32 channels ("a group") with one (C0 = 1) or two (C0 = 3) 32x32x16 MFMAs; what bounds it is
// the vector work around them, so the operands are laid out to need almost none:
//  * The window rows of a pixel lie in LDS as dwords (a row starts 16 or 32 bytes left of the tile's first window), and the
//    weights are permuted to the order in which they are read.  The matrix core rounds after each group of eight (a lane half's
//    operand), in which the order does not matter: the groups are those of k_conv0_fwd_tile, elements 0..7, 8..15, .. of the
//    9*C0 window values row after row, and the sums its sums, bit for bit.  (A network may have its policy step here and its
//    update there: the update's first step must see the policy that acted.)  C0 = 1: two dwords per row, (2x-2, 2x-1) and
//    (2x, 2x+1), packed so that lane half 0 has eight taps and half 1 the ninth: two permutes, four masks.  C0 = 3: five
//    dwords per row, the value in front of the window and its nine (x 0)(1 2)(3 4)(5 6)(7 8); a group is whole dwords and a pair
//    from two others.  The last dwords of rows 0 and 1, which the other lane half's groups take too, change halves in one swap:
//    nine dwords read, one swap, two permutes, two masks.  Values outside the window have zero weights and are masked
//    off as well: a NaN there must not reach the sum.
//  * The weights' rows are permuted so that a lane ends up with 16 consecutive channels of its pixel: 8 conversions, 8
//    clamps, two 16-byte LDS writes, and (BITS) its 16 mask bits are a half-word of the pixel's mask word.
//  * Pixel -> address is the same for every tile; only tiles at an image's edge test which pixels exist (the others are
//    written as zeros: the second layer's padding).
// About 30 vector instructions per group, 50 with the mask bits (some 150 in the kernel that writes the layer out).
// Measured (16384 images of 120x160, the layers' own kernels before -> this): forward 1206 + 1420 -> 1204 us (mask bits of both
// layers stored), weight gradient of the second layer 1124 -> 1271 us (1180 with the later changes to its waves); forward alone, 4096 images, 279 + 367 -> 279 us.  The
// rows are made at the expense of the compute waves' issue slots: matrix and vector instructions together fill 0.79 of a
// SIMD's cycles forward, 0.76 in the weight gradient; memory would allow some 860 and 650 us.
#pragma once
#include "conv_bits.hip.h"

// An LDS write behind the compiler's back: in front of an ordinary one it waits for every LDS-writing load of the wave, i.e.
// for the images that are to arrive several tiles later.  The caller waits (lgkmcnt) before the barrier that hands the row over.
__device__ __forceinline__ void lds_write16_untracked(char* p, uint32_t x, uint32_t y, uint32_t z, uint32_t w) {
  typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
  const u32x4_t v = {x, y, z, w};
  asm volatile("ds_write_b128 %0, %1" : : "v"((uint32_t)(uintptr_t)LDS_AS(p)), "v"(v) : "memory");
}

// wait until at most n (>= 0) of this wave's vector-memory operations are outstanding, or a few fewer: in the steady state one
// or two comparisons instead of the search among 64 exact counts
__device__ __forceinline__ void vm_wait_few(int n) {
  if (n >= 12) vm_wait<12>();
  else if (n >= 10) vm_wait<10>();
  else if (n >= 8) vm_wait<8>();
  else if (n >= 4) vm_wait<4>();
  else if (n >= 2) vm_wait<2>();
  else if (n == 1) vm_wait<1>();
  else vm_wait<0>();
}

struct Conv0Src {
  ImgAddr img;           // input images [H][rowbytes], gathered through idx
  const bf16_t* w;       // [32][9*C0]
  const float* bias;     // [32]
  uint32_t* bits;        // BITS: one word per pixel of the first layer's output, bit c = channel c is positive
  int H, rowbytes;       // rows of rowbytes = 2 * C0 * W bytes, a multiple of 16
  int bpitch;            // BITS: words per row
  int nimage;            // LDS slots of the image ring (bands in flight + 1)
};

template <int C0>
struct Conv0Shape1 {
  static constexpr int LEAD = C0 == 1 ? 1 : 2;             // 16-byte pieces of a row in front of image column 4*col0
  static constexpr int GPW = 5, MAXL = C0 == 1 ? 3 : 6;    // groups and image loads per producer wave and tile
  static constexpr int MAXPIX = 4 * GPW * 32;
  static constexpr int AHEAD = 3;                          // images in flight, if the LDS holds one more than that
  __host__ __device__ static int row_pitch(int TC) { return (LEAD * 16 + 8 * C0 * TC + 15) & ~15; }
  __host__ __device__ static int image_bytes(int TC, int TR) { return (4 * TR + 3) * row_pitch(TC) + 16; }  // (the last window row's reads may run 4 bytes over, 8 with three channels)
  __host__ __device__ static int act_bytes(int TC, int TR) { return ((2 * TR + 1) * (2 * TC + 1) * 64 + 64 + 127) & ~127; }  // ends in a pixel that takes what no pixel wants
  static bool fits(int TC, int TR) { return (4 * TR + 3) * row_pitch(TC) <= MAXL * 4096 && 4 * TR + 3 <= 255; }
};

// One of four producer waves.  Tile: TR x TC output pixels of the SECOND layer; its input rows 2*TR+1 of 2*TC+1 slots, slot 0 =
// column 2*col0 - 1.  COLS = false: the tile spans the image (TC = Wo, col0 = 0) and its pad slots are zeroed once by the caller.
template <int C0, bool COLS, bool BITS>
struct Conv0Producer {
  typedef Conv0Shape1<C0> S;
  static constexpr int KS = C0 == 1 ? 1 : 2, GPW = S::GPW, MAXL = S::MAXL;
  static constexpr int NOFF = C0 == 1 ? 1 : 2;
  int b1[GPW], dlt[NOFF], pitch, ng, nl;
  uint32_t wa[GPW], rc[GPW], boff[GPW];
  int goff[MAXL];
  uint32_t rs[MAXL];
  bf16x8_t w[KS];
  f32x16_t bias;
  uint32_t m2, m3, m4, negw[2];

  __device__ __forceinline__ void init(const Conv0Src& s, int aw, int lane, int TR, int TC, int W1) {
    const int l32 = lane & 31, h = lane >> 5, LB = S::row_pitch(TC), WP = 2 * TC + 1;
    const int ncol = COLS ? WP : W1, s0 = COLS ? 0 : 1, npx = (2 * TR + 1) * ncol, ngr = (npx + 31) >> 5;
    ng = (ngr - aw + 3) >> 2;
    pitch = LB;
    const int nbytes = (4 * TR + 3) * LB;
    nl = (((nbytes + 1023) >> 10) - aw + 3) >> 2;
#pragma unroll
    for (int i = 0; i < MAXL; ++i) {
      const int p = (aw + 4 * i) * 1024 + lane * 16, row = p / LB, in = p - row * LB;
      goff[i] = row * s.rowbytes + in - S::LEAD * 16;
      rs[i] = p < nbytes ? (uint32_t)row | (uint32_t)(in >> 4) << 8 : 0xffffffffu;
    }
#pragma unroll
    for (int g = 0; g < GPW; ++g) {
      int p = (aw + 4 * g) * 32 + l32;
      const bool live = p < npx;
      if (!live) p = 0;
      const int row = p / ncol, sl = s0 + p - row * ncol;
      b1[g] = 2 * row * LB + (C0 == 1 ? 8 + 4 * sl : 12 + 12 * sl);
      wa[g] = live ? (uint32_t)(row * WP * 64) + ((uint32_t)(sl * 64 + h * 32) ^ tile_swz_bits<32>((uint32_t)(sl * 64)))
                   : (uint32_t)((2 * TR + 1) * WP * 64 + h * 32);
      rc[g] = (uint32_t)row | (uint32_t)sl << 16;
      boff[g] = (uint32_t)(((row - 1) * s.bpitch + sl - 1) * 4 + h * 2);
    }
#pragma unroll
    for (int i = 0; i < NOFF; ++i) dlt[i] = C0 == 1 ? 2 * LB + 4 * h : i == 0 ? h * LB : 2 * LB + 12 * h;
    // row i of the product is channel ch: a lane's accumulators are then the channels h*16 .. h*16 + 15
    const int ch = ((l32 >> 2) & 1) * 16 + (l32 >> 3) * 4 + (l32 & 3);
    const bf16_t* wp = s.w + ch * 9 * C0;
    uint32_t v[8 * KS];
#pragma unroll
    for (int k = 0; k < 8 * KS; ++k) {
      // k-th value of this lane half: element t of window row u, or none
      int u, t;
      if (C0 == 1) { constexpr int order[8] = {0, 3, 1, 2, 4, 5, 6, 7}; u = 0; t = h ? (k == 6 ? 8 : -1) : order[k & 7]; }
      else if (k < 8) { u = k == 1 ? 0 : h; t = k == 1 ? 7 + h : k == 0 ? 0 : k - 1; }
      else if (k < 10) { u = 1; t = h ? -1 : k - 1; }
      else if (k < 12) { u = 2; t = h ? k - 3 : k - 9; }
      else { u = 2; t = k == 15 ? 5 + h : h ? -1 : k == 14 ? 0 : k - 9; }
      v[k] = t >= 0 ? (uint32_t)wp[t >= 0 ? u * 3 * C0 + t : 0] : 0u;
    }
#pragma unroll
    for (int m = 0; m < KS; ++m)
      w[m] = __builtin_bit_cast(bf16x8_t, make_uint4(v[8 * m] | v[8 * m + 1] << 16, v[8 * m + 2] | v[8 * m + 3] << 16, v[8 * m + 4] | v[8 * m + 5] << 16, v[8 * m + 6] | v[8 * m + 7] << 16));
#pragma unroll
    for (int e = 0; e < 16; ++e) bias[e] = s.bias[h * 16 + e];
    // C0 = 1: half 1 has but the first value of its shifted row; C0 = 3: the pairs (0 of row h, 7 or 8 of row 0) and (0 and 5 of
    // row 2, or 6 of row 2)
    m2 = h ? 0u : 0xffffffffu;
    m3 = C0 == 1 ? (h ? 0x0000ffffu : 0xffffffffu) : (h ? 0x07060302u : 0x05040302u);
    m4 = h ? 0x03020c0cu : 0x05040302u;
    negw[0] = nonzero_weights(0); negw[1] = nonzero_weights(1);
  }

  // Load i of this wave's loads of a tile's image rows; src: byte 8*C0*col0 of image row iy_lo, ix0 = that byte / 16
  struct Img { const char *src, *zp; char* dst; int iy_lo, H, ix0, pieces, aw; };
  __device__ __forceinline__ void load(const Img& m, int i) const {
    const int iy = m.iy_lo + (int)(rs[i] & 255u), ix = m.ix0 - S::LEAD + (int)(rs[i] >> 8);
    const char* p = ((uint32_t)iy < (uint32_t)m.H && (uint32_t)ix < (uint32_t)m.pieces) ? m.src + goff[i] : m.zp;
    if (rs[i] != 0xffffffffu) __builtin_amdgcn_global_load_lds(GLOBAL_AS(p), LDS_AS(m.dst + (m.aw + 4 * i) * 1024), 16, 0, 0);
  }
  __device__ __forceinline__ void load_all(const Img& m) const {
#pragma unroll
    for (int i = 0; i < MAXL; ++i)
      if (i < nl) load(m, i);
  }

  // This wave's groups of a tile (NG, at least ng: a group too many takes what it makes nowhere new); row_lo, col_lo: the first
  // layer's row and column of slot (0, 0); bits: the mask word of (row_lo + 1, col_lo + 1).  EDGE: the tile holds pixels outside
  // the image.  after(g): called behind group g.  All LDS reads come first and the sums run two groups ahead of the vector
  // work on them: the compute wave on the same SIMD leaves a lone dependent chain little.  Returns the stores surely issued.
  template <int NG, bool EDGE, class F>
  __device__ __forceinline__ int groups(const char* im, char* act, int row_lo, int col_lo, int H1, int W1, char* bits, F after) const {
    constexpr int ND = C0 == 1 ? 6 : 9;
    uint32_t d[NG][ND];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const char* const p1 = im + b1[g];
#pragma unroll
      for (int i = 0; i < ND; ++i) {
        // C0 = 3: 0..4 = row h, 5..8 = row 2 from its first dword, or from (5 6) on in half 1 (whose last two are nobody's)
        const char* p = C0 == 1 ? (i < 2 ? p1 : i < 4 ? p1 + pitch : p1 + dlt[0]) + 4 * (i & 1) : i < 5 ? p1 + dlt[0] + 4 * i : p1 + dlt[NOFF - 1] + 4 * (i - 5);
        d[g][i] = *reinterpret_cast<const uint32_t*>(p);
      }
      // three channels: group after group, so that the first sums wait for few of the 45 reads (8192 stereo pairs: weight gradient
      // 1667 -> 1624 us, forward 1381 -> 1298)
      if (C0 > 1) __builtin_amdgcn_sched_barrier(0);
    }
    auto sums = [&](int g) __attribute__((always_inline)) {
      const uint32_t* const x = d[g];
      if constexpr (C0 == 1) {
        const uint4 v = make_uint4(__builtin_amdgcn_perm(x[2], x[0], 0x07060302u) & m2, x[1] & m2, x[3] & m2, __builtin_amdgcn_alignbit(x[5], x[4], 16) & m3);
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[0], __builtin_bit_cast(bf16x8_t, v), bias, 0, 0, 0);
      } else {
        // (dwords stand where the pairs of reads put them: no moves)
        const auto last = __builtin_amdgcn_permlane32_swap(x[4], x[4], false, false);  // of row 0, of row 1, in both halves
        const uint4 u = make_uint4(__builtin_amdgcn_perm(last[0], x[0], m3), x[1], x[2], x[3]);
        const f32x16_t acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[0], __builtin_bit_cast(bf16x8_t, u), bias, 0, 0, 0);
        const uint4 v = make_uint4(last[1] & m2, x[6], x[7] & m2, __builtin_amdgcn_perm(x[8], x[5], m4));
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[KS - 1], __builtin_bit_cast(bf16x8_t, v), acc, 0, 0, 0);
      }
    };
    f32x16_t acc[3];
#pragma unroll
    for (int g = 0; g < 2 && g < NG; ++g) acc[g] = sums(g);
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      if (g + 2 < NG) acc[(g + 2) % 3] = sums(g + 2);
      __builtin_amdgcn_sched_barrier(0);
      const f32x16_t& cur = acc[g % 3];
      uint32_t o[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = relu_pack2bf(cur[2 * e], cur[2 * e + 1]);
      bool ok = true;
      if constexpr (EDGE) {
        const int y = row_lo + (int)(rc[g] & 0xffffu), x = col_lo + (int)(rc[g] >> 16);
        ok = (uint32_t)y < (uint32_t)H1 && (uint32_t)x < (uint32_t)W1;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = ok ? o[e] : 0u;
      }
      lds_write16_untracked(act + wa[g], o[0], o[1], o[2], o[3]);
      lds_write16_untracked(act + (wa[g] ^ 16u), o[4], o[5], o[6], o[7]);
      if constexpr (BITS) {
        uint32_t b[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const uint32_t s0 = nonzero_signs(o[4 * q], o[4 * q + 1]), s1 = nonzero_signs(o[4 * q + 2], o[4 * q + 3]);
          b[q] = (uint32_t)__builtin_amdgcn_sdot4((int)s1, (int)negw[1], __builtin_amdgcn_sdot4((int)s0, (int)negw[0], 0, false), false);
        }
        // (pixels of the rows and columns that a neighbouring tile makes too are stored by both, alike)
        if (ok) *reinterpret_cast<unsigned short*>(bits + (int)boff[g]) = (unsigned short)(b[0] | b[1] << 8);
      }
      after(g);
    }
    return BITS && !EDGE ? NG : 0;
  }
  template <class F>
  __device__ __forceinline__ int produce(const char* im, char* act, bool edge, int row_lo, int col_lo, int H1, int W1, char* bits, F after) const {
    if (ng > 3) return edge ? groups<GPW, true>(im, act, row_lo, col_lo, H1, W1, bits, after) : groups<GPW, false>(im, act, row_lo, col_lo, H1, W1, bits, after);
    return edge ? groups<3, true>(im, act, row_lo, col_lo, H1, W1, bits, after) : groups<3, false>(im, act, row_lo, col_lo, H1, W1, bits, after);
  }
};
