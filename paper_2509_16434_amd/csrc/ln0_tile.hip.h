// First convolution (one-channel images, 16 output channels, 3x3 stride 2 pad 1), layer normalisation over the image and ReLU in
// one kernel, and the backward of the three - gradients of gain, shift, weights and bias - in another.  The convolution's output
// and its gradient, 16 times the image's pixels / 4, are the teacher's largest tensors: they stay in the registers of the block
// that makes an image (a few products of depth 9 per value), the backward pass makes them again from the image.  What is left to
// move is the image, the rectified output (forward) and its gradient (backward).
//
// A block of eight waves takes one image at a time.  A tile is 16 pixels x 16 channels, one 16x16x32 MFMA (9 of 32 deep; the thin
// product costs less than any other way to gather the windows); a wave has the tiles wave, wave + 8, .. of the image, at most NT.
//  * The image lies in LDS as three planes per row, plane v = the pixels 2x-1+v: a tap is then a constant offset, and a
//    transposing read hands a lane four taps of its pixel.
//  * A lane holds channels 4*(lane/16) .. + 3 of pixel lane%16 of each of its tiles, rounded to bf16 as a stored output would be:
//    8 bytes to load (gradient) or store (output).
//  * Weight gradient: the pixels' gradients pass through a strip of LDS (8 bytes written per lane, one transposing read) to become
//    the operand of a product over 32 pixels; its other operand, the windows, is 16 neighbouring bytes of two planes' rows.
//  * The next image's pixels, and backward its gradient tile by tile as this image's is consumed, are on their way in registers.
// Backward is bound by vector issue: some hundred instructions per tile fill 0.83 of its SIMDs' cycles.  Forward by neither issue
// (0.56) nor memory alone (800 MB at 3.6 TB/s, of which 629 are stores): an image's stores follow its sums, and one block is all
// that a CU's registers hold.  4096 images of 120x160, with the layer's kernels before (convolution, normalisation; their
// backward): forward 169 + 234 -> 219 us, backward 376 + 157 -> 265 to 277.
#pragma once
#include "conv_small.hip.h"
#include "recurrent.hip.h"

struct Ln0Args {
  ImgAddr in;              // images [H][W], gathered through idx; W a multiple of 8
  const bf16_t* w;         // [16][9]
  const float *bias, *gain, *shift;
  int nimg, H, W, Ho, Wo;
  FastDiv w4;              // division by W / 8 (at least 2): groups of four output pixels per row
  float2* stats;           // (mean, rstd) per image: written forward, read backward
  ImgAddrW out;            // forward: rectified output [Ho][Wo][16]
  int P;                   // forward: the proprioception's columns of the feature rows
  const bf16_t* proprio;
  bf16_t* feat;
  int64_t feat_ld;
  ImgAddr dy;              // backward: gradient of the output (need not be masked)
  float *part_ln, *part_w; // backward, per block: [32] gain and shift gradients, [16][10] weight and bias gradients
};
struct Ln0Shape {
  static constexpr int THREADS = 512, NW = 8, ICH = 5, MAXNT = 38;  // ICH: 16-byte pieces of an image per thread
  __host__ __device__ static int row_bytes(int W) { return 3 * W; }   // three planes of W / 2 pixels
  __host__ __device__ static int plane_bytes(int Ho, int W) { return (2 * Ho + 1) * row_bytes(W); }
  static constexpr int CONST_BYTES = 32;                              // zeros, ones
  static constexpr int RED_BYTES = 2 * 2 * NW * 4;
  static int lds_bytes(int Ho, int W, bool bwd) {
    const int n = ((2 * plane_bytes(Ho, W) + 15) & ~15) + CONST_BYTES + RED_BYTES + (bwd ? NW * 1024 : 0), sums = NW * (256 + 32) * 4;
    return bwd && n < sums ? sums : n;
  }
  static int tiles(int Ho, int W) { return (Ho * (W / 2) + 15) / 16; }
  static bool covers(int H, int W, int Ho) {
    return W >= 16 && tiles(Ho, W) <= NW * MAXNT && lds_bytes(Ho, W, true) <= 160 * 1024 && H * (W / 8) <= ICH * THREADS;
  }
};
// What both directions share.  Pixels are numbered with the rows rounded up to multiples of four (W / 2 slots); RAG: some of them
// are no pixels.
template <bool RAG>
struct Ln0Image {
  char *planes, *zero;  // of the current image; zeros, then ones
  int rb, rowstep, np4, slots, tid, l16, q;
  uint32_t m0, m1, o0, o1;
  bf16x8_t w;
  cs_f4 bias;
  uint4 px[Ln0Shape::ICH];

  __device__ __forceinline__ void init(const Ln0Args& a, char* lds, int total) {
    tid = threadIdx.x;
    const int lane = tid & 63;
    l16 = lane & 15; q = lane >> 4;
    rb = Ln0Shape::row_bytes(a.W); rowstep = 2 * rb - a.W; slots = a.W >> 1; np4 = a.Ho * (a.W >> 3);
    for (int i = tid; i < total / 16; i += Ln0Shape::THREADS) reinterpret_cast<uint4*>(lds)[i] = make_uint4(0u, 0u, 0u, 0u);
    // transposing reads: lane (q, r) supplies pixels 4 (r & 3) .. of tap r >> 2 (+ 4) for q = 0, of tap 8 for q = 1
    const int tap0 = q == 0 ? l16 >> 2 : (q == 1 && (l16 >> 2) == 0) ? 8 : -1, tap1 = q == 0 ? (l16 >> 2) + 4 : -1;
    auto off = [&](int t) { return (uint32_t)((t / 3) * rb + (t % 3) * a.W); };
    m0 = tap0 >= 0 ? ~0u : 0u; m1 = tap1 >= 0 ? ~0u : 0u;
    o0 = tap0 >= 0 ? off(tap0) : 0u; o1 = tap1 >= 0 ? off(tap1) : 0u;
    uint32_t v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = q == 0 ? (uint32_t)a.w[l16 * 9 + k] : (q == 1 && k == 0) ? (uint32_t)a.w[l16 * 9 + 8] : 0u;
    w = __builtin_bit_cast(bf16x8_t, make_uint4(v[0] | v[1] << 16, v[2] | v[3] << 16, v[4] | v[5] << 16, v[6] | v[7] << 16));
#pragma unroll
    for (int i = 0; i < 4; ++i) bias[i] = a.bias[q * 4 + i];
  }
  __device__ __forceinline__ void fetch(const Ln0Args& a, int img) {
    const bf16_t* const p = a.in.ptr_uniform(img);
    const int n = a.H * (a.W >> 3);
#pragma unroll
    for (int j = 0; j < Ln0Shape::ICH; ++j) px[j] = *reinterpret_cast<const uint4*>(p + (int64_t)min((int)threadIdx.x + j * Ln0Shape::THREADS, n - 1) * 8);
  }
  // the fetched image into its planes; rows above and below it and the column left of it stay zero
  __device__ __forceinline__ void put(const Ln0Args& a, char* dst) const {
    const int n = a.H * (a.W >> 3), W4 = a.W >> 3;
#pragma unroll
    for (int j = 0; j < Ln0Shape::ICH; ++j) {
      const int i = tid + j * Ln0Shape::THREADS;
      if (i < n) {
        const int r = (int)a.w4.div2((uint32_t)i), c = i - r * W4;
        char* const p = dst + (r + 1) * rb + c * 8;
        const uint4 v = px[j];
        const uint32_t e0 = __builtin_amdgcn_perm(v.y, v.x, 0x05040100u), e1 = __builtin_amdgcn_perm(v.w, v.z, 0x05040100u);  // pixels 0 2, 4 6
        const uint32_t d0 = __builtin_amdgcn_perm(v.y, v.x, 0x07060302u), d1 = __builtin_amdgcn_perm(v.w, v.z, 0x07060302u);  // pixels 1 3, 5 7
        *reinterpret_cast<uint2*>(p + a.W) = make_uint2(e0, e1);
        *reinterpret_cast<uint2*>(p + 2 * a.W) = make_uint2(d0, d1);
        *reinterpret_cast<unsigned short*>(p + 2) = (unsigned short)d0;
        *reinterpret_cast<uint32_t*>(p + 4) = __builtin_amdgcn_alignbit(d1, d0, 16);
        if (c + 1 < W4) *reinterpret_cast<unsigned short*>(p + 8) = (unsigned short)(d1 >> 16);
      }
    }
  }
  // byte offset of the four pixels p4 in plane 0 of the row above theirs
  __device__ __forceinline__ uint32_t at(const Ln0Args& a, int p4) const {
    const int p = min(p4, np4 - 1);
    return (uint32_t)(p * 8 + (int)a.w4.div2((uint32_t)p) * rowstep);
  }
  // bf16 pairs of this lane's four channels of its pixel of tile t
  __device__ __forceinline__ uint2 conv(const Ln0Args& a, int t) const {
    const uint32_t b = at(a, 4 * t + (l16 & 3));
    const char* const p0 = m0 ? planes + o0 + b : zero;
    const char* const p1 = m1 ? planes + o1 + b : zero;
    const cs_f4 d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, lds_read_tr8_2(p0, p1), bias, 0, 0, 0);
    return make_uint2(pack2bf(d[0], d[1]), pack2bf(d[2], d[3]));
  }
  // does the lane's pixel of tile t exist, and its byte offset in the output (beyond it, if not)
  __device__ __forceinline__ bool exists(const Ln0Args& a, int t, uint32_t* off) const {
    const int p = 16 * t + l16;
    if constexpr (RAG) {
      const int y = (int)a.w4.div2((uint32_t)(p >> 2)), x = p - y * slots;
      const bool ok = y < a.Ho && x < a.Wo;
      *off = ok ? (uint32_t)((y * a.Wo + x) * 32 + q * 8) : 0x7ffffff0u;
      return ok;
    } else {
      *off = (uint32_t)(p * 32 + q * 8);
      return p < a.Ho * a.Wo;
    }
  }
};
// sums of x and y over the block, in a fixed order; red: [2][8], another one at the next call
__device__ __forceinline__ float2 ln0_block_sum(float x, float y, float* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) { x += __shfl_xor(x, off); y += __shfl_xor(y, off); }
  if ((threadIdx.x & 63) == 0) { red[threadIdx.x >> 6] = x; red[8 + (threadIdx.x >> 6)] = y; }
  __syncthreads();
  float sx = 0.f, sy = 0.f;
#pragma unroll
  for (int w = 0; w < 8; ++w) { sx += red[w]; sy += red[8 + w]; }
  return make_float2(sx, sy);
}
__device__ __forceinline__ void unpack4(const uint2& u, float (&f)[4]) {
  f[0] = __uint_as_float(u.x << 16); f[1] = __uint_as_float(u.x & 0xffff0000u);
  f[2] = __uint_as_float(u.y << 16); f[3] = __uint_as_float(u.y & 0xffff0000u);
}
typedef uint32_t u32x2_buf_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t ln0_rsrc(const bf16_t* p, uint32_t bytes) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p), 0, bytes, 0x00027000); }

template <int NT, bool RAG>
__global__ __launch_bounds__(512) void k_conv0_ln_fwd(Ln0Args a) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  typedef Ln0Shape S;
  const int pb = S::plane_bytes(a.Ho, a.W), total = (2 * pb + 15) & ~15;
  Ln0Image<RAG> im;
  im.fetch(a, blockIdx.x);
  im.init(a, lds, total + S::CONST_BYTES);
  im.zero = lds + total;
  float* const red = reinterpret_cast<float*>(lds + total + S::CONST_BYTES);
  __syncthreads();
  im.put(a, lds);
  const int wave0 = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), m = a.Ho * a.Wo * 16;
  float gain[4], shift[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) { gain[i] = a.gain[im.q * 4 + i]; shift[i] = a.shift[im.q * 4 + i]; }
  int par = 0;
  for (int img = blockIdx.x; img < a.nimg; img += gridDim.x, par ^= 1) {
    __syncthreads();  // the image's planes are written; red may be written again
    im.planes = lds + par * pb;
    int wave = wave0;
    asm volatile("" : "+s"(wave));  // (the tiles' addresses are not to be kept from image to image: they are more than the registers)
    const int next = img + (int)gridDim.x < a.nimg ? img + (int)gridDim.x : img;  // (the last one is fetched again: no branch)
    im.fetch(a, next);
    if (img % a.in.V == 0) {
      const int b = img / a.in.V;
      const int64_t sm = a.in.idx ? a.in.idx[b] : b;
      for (int i = im.tid; i < a.P >> 3; i += S::THREADS) reinterpret_cast<uint4*>(a.feat + (int64_t)b * a.feat_ld)[i] = reinterpret_cast<const uint4*>(a.proprio + sm * a.P)[i];
    }
    uint2 x[NT];
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      x[j] = im.conv(a, wave + 8 * j);
      uint32_t off;
      const bool ok = im.exists(a, wave + 8 * j, &off);
      float f[4];
      unpack4(x[j], f);
      s += ok ? (f[0] + f[1]) + (f[2] + f[3]) : 0.f;
      asm volatile("" : "+v"(x[j].x), "+v"(x[j].y));
      __builtin_amdgcn_sched_barrier(0);
    }
    const float mean = ln0_block_sum(s, 0.f, red).x / (float)m;
    asm volatile("" : "+s"(wave));
    float v = 0.f;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      uint32_t off;
      const bool ok = im.exists(a, wave + 8 * j, &off);
      float f[4];
      unpack4(x[j], f);
      float d = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) { const float e = f[i] - mean; d += e * e; }
      v += ok ? d : 0.f;
      asm volatile("" : "+v"(x[j].x), "+v"(x[j].y));
    }
    const float rstd = rsqrtf(ln0_block_sum(v, 0.f, red + 16).x / (float)m + LN_EPS);
    if (im.tid == 0) a.stats[img] = make_float2(mean, rstd);
    float g[4], b[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) { g[i] = gain[i] * rstd; b[i] = shift[i] - mean * g[i]; }
    asm volatile("" : "+s"(wave));
    const auto ro = ln0_rsrc(a.out.ptr(img), (uint32_t)m * 2u);
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      uint32_t off;
      im.exists(a, wave + 8 * j, &off);  // (the hardware drops stores beyond the image)
      float f[4];
      unpack4(x[j], f);
      float y[4];  // (of a non-finite image: zeros, as k_ln_fwd leaves them)
#pragma unroll
      for (int i = 0; i < 4; ++i) y[i] = fmaxf(f[i] * g[i] + b[i], 0.f);
      const u32x2_buf_t o = {pack2bf(y[0], y[1]), pack2bf(y[2], y[3])};
      __builtin_amdgcn_raw_buffer_store_b64(o, ro, off, 0, 0);
    }
    im.put(a, lds + (par ^ 1) * pb);
  }
}

template <int NT, bool RAG>
__global__ __launch_bounds__(512) void k_conv0_ln_bwd(Ln0Args a) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  typedef Ln0Shape S;
  const int pb = S::plane_bytes(a.Ho, a.W), total = (2 * pb + 15) & ~15;
  Ln0Image<RAG> im;
  im.fetch(a, blockIdx.x);
  im.init(a, lds, total + S::CONST_BYTES);
  im.zero = lds + total;
  char* const ones = im.zero + 16;
  float* const red = reinterpret_cast<float*>(lds + total + S::CONST_BYTES);
  const int wave0 = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), m = a.Ho * a.Wo * 16;
  char* const strip = lds + total + S::CONST_BYTES + S::RED_BYTES + wave0 * 1024;
  __syncthreads();
  if (im.tid < 4) reinterpret_cast<uint32_t*>(ones)[im.tid] = 0x3F803F80u;
  im.put(a, lds);
  const int l16 = im.l16, q = im.q;
  float dg[4], db[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) { dg[i] = 0.f; db[i] = 0.f; }
  // the windows as operand: column l16 is tap l16 (9: ones, beyond: zeros) of the pixels 4q .. + 3 of two tiles
  const uint32_t tapoff = l16 < 9 ? (uint32_t)((l16 / 3) * im.rb + (l16 % 3) * a.W) : 0u;
  const char* const fixed = l16 == 9 ? ones : im.zero;
  char* const sw = strip + l16 * 32 + q * 8;                                    // this lane's 8 bytes of a tile
  const char* const sr = strip + (q * 4 + (l16 >> 2)) * 32 + (l16 & 3) * 8;      // its part of the transposing read
  cs_f4 wacc = {0.f, 0.f, 0.f, 0.f};
  uint2 dv[NT];
  auto load_dy = [&](__amdgpu_buffer_rsrc_t rd, int j, int wave) __attribute__((always_inline)) {
    uint32_t off;
    im.exists(a, wave + 8 * j, &off);  // (zeros beyond the image)
    dv[j] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(rd, off, 0, 0));
  };
  auto dy_of = [&](int img) { return ln0_rsrc(a.dy.ptr_uniform(img), (uint32_t)m * 2u); };
  {
    const auto rd = dy_of(blockIdx.x);
#pragma unroll
    for (int j = 0; j < NT; ++j) load_dy(rd, j, wave0);
  }
  int par = 0;
  for (int img = blockIdx.x; img < a.nimg; img += gridDim.x, par ^= 1) {
    __syncthreads();  // the image's planes are written
    im.planes = lds + par * pb;
    int wave = wave0;
    asm volatile("" : "+s"(wave));  // (the tiles' addresses are not to be kept from image to image: they are more than the registers)
    const int next = img + (int)gridDim.x < a.nimg ? img + (int)gridDim.x : img;  // (the last one is fetched again: no branch)
    const auto rdn = dy_of(next);
    const float2 st = a.stats[img];
    const float rstd = st.y, mr = st.x * rstd;
    float gr[4], br[4];  // the forward's y = x * gr + br
    int c0 = q * 4;
    asm volatile("" : "+v"(c0));  // (gains and shifts are read for each image: there is no register to spare)
#pragma unroll
    for (int i = 0; i < 4; ++i) { gr[i] = a.gain[c0 + i] * rstd; br[i] = a.shift[c0 + i] - st.x * gr[i]; }
    uint2 x[NT];
    float s1 = 0.f, s2 = 0.f;  // sums of dxhat * rstd and of that times xhat
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      x[j] = im.conv(a, wave + 8 * j);
      float f[4], d[4];
      unpack4(x[j], f); unpack4(dv[j], d);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float dj = f[i] * gr[i] + br[i] > 0.f ? d[i] : 0.f, xh = f[i] * rstd - mr, dxh = dj * gr[i];
        s1 += dxh; s2 += dxh * xh;
        dg[i] += dj * xh; db[i] += dj;
      }
      // (not to be kept as floats for the second pass, nor the sums' updates to be put off until then)
      asm volatile("" : "+v"(x[j].x), "+v"(x[j].y), "+v"(dv[j].x), "+v"(dv[j].y));
#pragma unroll
      for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(dg[i]), "+v"(db[i]));
      __builtin_amdgcn_sched_barrier(0);
    }
    const float2 sums = ln0_block_sum(s1, s2, red + par * 16);
    const float a1 = sums.x / (float)m, a2 = sums.y / (float)m, xs = -a2 * rstd, xc = a2 * mr - a1;  // dx = dj * gr - (a1 + xhat a2)
    im.fetch(a, next);
    asm volatile("" : "+s"(wave));
#pragma unroll
    for (int j = 0; j < NT; j += 2) {
      bf16x8_t av, bv;
      struct { uint2 t[2]; } bq;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        uint2 o = make_uint2(0u, 0u);
        bq.t[k] = o;
        if (j + k < NT) {
          const int t = wave + 8 * (j + k < NT ? j + k : 0);
          float f[4], d[4], r[4];
          const uint2 xj = x[j + k < NT ? j + k : 0], dj2 = dv[j + k < NT ? j + k : 0];
          unpack4(xj, f); unpack4(dj2, d);
#pragma unroll
          for (int i = 0; i < 4; ++i) r[i] = (f[i] * gr[i] + br[i] > 0.f ? d[i] : 0.f) * gr[i] + (f[i] * xs + xc);
          uint32_t off;
          const bool ok = im.exists(a, t, &off);
          o.x = ok ? pack2bf(r[0], r[1]) : 0u; o.y = ok ? pack2bf(r[2], r[3]) : 0u;
          const uint32_t b = im.at(a, 4 * t + q);
          bq.t[k] = *reinterpret_cast<const uint2*>(l16 < 9 ? im.planes + tapoff + b : fixed);
          if (j + k < NT) load_dy(rdn, j + k < NT ? j + k : 0, wave);
        }
        *reinterpret_cast<uint2*>(sw + k * 512) = o;
      }
      av = lds_read_tr8_2(sr, sr + 512);
      bv = __builtin_bit_cast(bf16x8_t, bq);
      wacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, wacc, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    im.put(a, lds + (par ^ 1) * pb);
  }
  // ---- this block's sums: over the 16 pixels of a lane group, then over the waves
#pragma unroll
  for (int off = 1; off < 16; off <<= 1)
#pragma unroll
    for (int i = 0; i < 4; ++i) { dg[i] += __shfl_xor(dg[i], off); db[i] += __shfl_xor(db[i], off); }
  __syncthreads();
  float* const R = reinterpret_cast<float*>(lds);  // [wave][16][16] weight gradients, then [wave][32]
  float* const RL = R + 8 * 256;
#pragma unroll
  for (int i = 0; i < 4; ++i) R[wave0 * 256 + (q * 4 + i) * 16 + l16] = wacc[i];
  if (l16 == 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) { RL[wave0 * 32 + q * 4 + i] = dg[i]; RL[wave0 * 32 + 16 + q * 4 + i] = db[i]; }
  }
  __syncthreads();
  if (im.tid < 160) {
    const int ch = im.tid / 10, k = im.tid - ch * 10;
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < 8; ++w) s += R[w * 256 + ch * 16 + k];
    a.part_w[(int64_t)blockIdx.x * 160 + im.tid] = s;
  } else if (im.tid >= 192 && im.tid < 224) {
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < 8; ++w) s += RL[w * 32 + im.tid - 192];
    a.part_ln[(int64_t)blockIdx.x * 32 + im.tid - 192] = s;
  }
}
