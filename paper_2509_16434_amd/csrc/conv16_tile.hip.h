// 3x3 stride-2 pad-1 convolution from 16 to 32 channels: weight gradient and (unmasked) input gradient on LDS images of bands of
// whole rows.  (The forward is k_conv_fwd_tile<16>.)  All three are bound by memory: the 16-channel tensor, of four times the
// pixels, is two thirds of their bytes, which move at 5.1 to 6.1 TB/s while vector instructions fill at most 0.17 and products
// 0.14 of the cycles.  The implicit-GEMM kernels that such a layer took before gathered its windows through
// integer divisions at two thirds of that rate: 4096 images of 60x80, forward 245 -> 180 us, input gradient
// 266 -> 196, weight gradient 274 -> 156.
#pragma once
#include "conv_dgrad_tile.hip.h"
#include "conv_small.hip.h"

// Weight gradient.  Four loader waves and four compute waves on a ring of bands, as in k_conv_wgrad_tile; the compute waves share
// a band's pixels: wave w has the steps of 16 pixels w, w + 4, .. and all of the sum, G[n][k] with k = tap*16 + ci in five
// k-tiles of two taps each, whose tenth tap reads ones (the bias gradient).  A lane's tap of a tile is that of its half of the
// 32 columns.  The waves' sums are added in LDS at the end, in wave order.
struct Conv16WgradShape {
  static constexpr int PIX = 32, DY = 64, MAXSTEP = 16, MAXSEG = 6, MAXBUF = 6, THREADS = 512, KT = 5;
  __host__ __device__ static int image_bytes(int W, int TR) { return ((2 * TR + 1) * (W + 2) * PIX + 127) & ~127; }
  __host__ __device__ static int buf_bytes(int W, int TR, int nstep) { return image_bytes(W, TR) + nstep * 16 * DY; }
  static int lds_bytes(int W, int TR, int nstep, int nbuf) {
    const int n = nbuf * buf_bytes(W, TR, nstep) + 16, sums = 4 * KT * 16 * 64 * 4;
    return n < sums ? sums : n;
  }
};
__global__ __launch_bounds__(512) void k_conv16_wgrad_tile(ConvWgradArgs a) {
  typedef Conv16WgradShape S;
  constexpr int PIX = S::PIX, KT = S::KT;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int W = a.W, TR = a.TR, Wo = a.Wo, WP = W + 2, nstep = a.nstep, NBUF = a.nbuf, nrows = 2 * TR + 1;
  const int rowbytes = W * PIX, segs = (rowbytes + 1023) >> 10, image_bytes = S::image_bytes(W, TR), buf_bytes = S::buf_bytes(W, TR, nstep);
  const int vb = xcd_block((int)blockIdx.x, (int)gridDim.x);
  const int nq = (a.ntiles > vb) ? (a.ntiles - 1 - vb) / (int)gridDim.x + 1 : 0;
  char* const ones = lds + NBUF * buf_bytes;
  // the pixels left and right of every row are zeros
  for (int i = tid; i < NBUF * nrows * 4; i += S::THREADS) {
    const int chunk = i & 1, side = (i >> 1) & 1, row = i >> 2, b = row / nrows, rr = row - b * nrows;
    *reinterpret_cast<uint4*>(lds + b * buf_bytes + rr * WP * PIX + (side ? (W + 1) * PIX : 0) + chunk * 16) = make_uint4(0u, 0u, 0u, 0u);
  }
  if (tid < 4) reinterpret_cast<uint32_t*>(ones)[tid] = 0x3F803F80u;
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // before this wave's first barrier
  f32x16_t acc[KT];
#pragma unroll
  for (int t = 0; t < KT; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;

  if (wave >= 4) {
    // ------------------------------------------------------------------ loaders: rows lw, lw + 4, .. and 1 KiB pieces of dY
    const int lw = wave - 4;
    const int ni = ((nrows - lw + 3) >> 2) * segs + ((nstep - lw + 3) >> 2);
    const char* const zp = reinterpret_cast<const char*>(a.zpage) + lane * 16;
    int slot = 0;
    auto issue = [&](int q) {
      const int t = vb + q * gridDim.x, img = (int)a.dv_nb.div((uint32_t)t), band = t - img * a.NB, iy_lo = 2 * band * TR - 1;
      const char* xsrc = reinterpret_cast<const char*>(a.in.ptr_uniform(img)) + (int64_t)iy_lo * rowbytes;
      const char* dsrc = reinterpret_cast<const char*>(a.dy.ptr_uniform(img) + (int64_t)band * TR * Wo * a.Cout);
      const int plim = min(TR, a.Ho - band * TR) * Wo;
      char* buf = lds + slot * buf_bytes;
      slot = slot + 1 == NBUF ? 0 : slot + 1;
      for (int row = lw; row < nrows; row += 4) {
        const bool inside = iy_lo + row >= 0 && iy_lo + row < a.H;
#pragma unroll
        for (int sg = 0; sg < S::MAXSEG; ++sg)
          if (sg < segs) {
            const int o = sg * 1024 + lane * 16;
            const char* p = inside ? xsrc + (int64_t)row * rowbytes + o : zp;
            if (o < rowbytes) __builtin_amdgcn_global_load_lds(GLOBAL_AS(p), LDS_AS(buf + (row * WP + 1) * PIX + sg * 1024), 16, 0, LOAD_NT);
          }
      }
      for (int j = lw; j < nstep; j += 4) {  // 16 pixels of 64 bytes
        const int o = j * 1024 + lane * 16, p_ = o >> 6, cb = o & 63;
        const char* p = (p_ < plim && (cb >> 1) < a.Cout) ? dsrc + (int64_t)p_ * a.Cout * 2 + cb : zp;
        __builtin_amdgcn_global_load_lds(GLOBAL_AS(p), LDS_AS(buf + image_bytes + j * 1024), 16, 0, LOAD_NT);
      }
    };
    const int D = NBUF - 1;
    for (int q = 0; q < D && q < nq; ++q) issue(q);
    for (int q = 0; q < nq; ++q) {
      vm_wait_dyn(min(D - 1, nq - 1 - q) * ni);
      __builtin_amdgcn_s_barrier();
      if (q + D < nq) issue(q + D);
    }
  } else {
    // ------------------------------------------------------------------ compute waves
    const int g = lane >> 4, r16 = lane & 15;
    uint32_t xb[4][2], db[4][2];  // of the wave's steps, pixels +0..3 and +4..7 of the lane's group
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        int p = (wave + 4 * s) * 16 + 8 * (g >> 1) + (r16 >> 2) + 4 * hf;
        db[s][hf] = (uint32_t)(image_bytes + p * S::DY + (16 * (g & 1) + 4 * (r16 & 3)) * 2);
        if (p >= TR * Wo) p = 0;  // its dY is zero
        const int oyl = p / Wo, ox = p - oyl * Wo;
        xb[s][hf] = (uint32_t)((2 * oyl * WP + 2 * ox) * PIX + (r16 & 3) * 8);
      }
    uint32_t tapc[KT];
#pragma unroll
    for (int t = 0; t < KT; ++t) { const int tap = 2 * t + (g & 1); tapc[t] = (uint32_t)(((tap / 3) * WP + tap % 3) * PIX); }
    const bool one = (g & 1) != 0;  // of the last k-tile: the tenth tap
    int slot = 0;
    for (int q = 0; q < nq; ++q) {
      __builtin_amdgcn_s_barrier();  // band q is in LDS
      const char* buf = lds + slot * buf_bytes;
      slot = slot + 1 == NBUF ? 0 : slot + 1;
#pragma unroll
      for (int s = 0; s < 4; ++s)
        if (wave + 4 * s < nstep) {
          const bf16x8_t av = lds_read_tr8_2(buf + db[s][0], buf + db[s][1]);
          bf16x8_t bv[KT];
#pragma unroll
          for (int t = 0; t < KT; ++t) {
            const char *p0 = buf + xb[s][0] + tapc[t], *p1 = buf + xb[s][1] + tapc[t];
            if (t == KT - 1) { p0 = one ? ones : p0; p1 = one ? ones : p1; }
            bv[t] = lds_read_tr8_2(p0, p1);
          }
#pragma unroll
          for (int t = 0; t < KT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv[t], acc[t], 0, 0, 0);
        }
    }
  }
  __syncthreads();  // the ring is free
  float* const R = reinterpret_cast<float*>(lds);  // [wave][k-tile][accumulator][lane]
  if (wave < 4) {
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) R[((wave * KT + t) * 16 + e) * 64 + lane] = acc[t][e];
  }
  __syncthreads();
  // acc[t][e] = G[n][k] with k = 32 t + lane % 32, n = (e/4)*8 + (lane/32)*4 + e%4; stored k-major
  float* const P = a.partial + (int64_t)blockIdx.x * 144 * a.Cout;
  for (int i = tid; i < 145 * 32; i += S::THREADS) {
    const int k = i >> 5, n = i & 31, o = ((k >> 5) * 16 + (n >> 3) * 4 + (n & 3)) * 64 + (k & 31) + 32 * ((n >> 2) & 1);
    if (n >= a.Cout) continue;
    const float s = (R[o] + R[KT * 1024 + o]) + (R[2 * KT * 1024 + o] + R[3 * KT * 1024 + o]);
    if (k < 144) P[k * a.Cout + n] = s;
    else if (a.bias_partial) a.bias_partial[(int64_t)blockIdx.x * a.Cout + n] = s;
  }
}

// Input gradient, from 32 channels to 16: quads (2x2 pixels of the result, conv_dgrad_tile.hip.h) are the columns of nine 16x16x32
// products, one per tap, whose depth is the 32 gradient channels.  Blocks of four waves, four to a CU, each load, multiply and
// write out a band in turn: what one waits for the others fill.  The result is staged in LDS and leaves as 16-byte pieces of the
// band's contiguous rows.  The 16-byte pieces of a dY pixel are permuted by its slot / 4, so that eight lanes' reads of eight
// neighbouring pixels fall into different banks.
struct Conv16DgradShape {
  static constexpr int CI = 16, CO = 32, BQ = 128, THREADS = 256, MAXSEG = 8;
  __host__ __device__ static int dyimg_bytes(int Wo, int TQ) { return (TQ + 1) * (Wo + 1) * 64; }
  __host__ __device__ static int stage_bytes(int W, int TQ) { return 2 * TQ * W * 32; }
  static int lds_bytes(int W, int Wo, int TQ) { return 2 * dyimg_bytes(Wo, TQ) + stage_bytes(W, TQ); }
};
__global__ __launch_bounds__(256, 4) void k_conv16_dgrad_tile(ConvDgradArgs a) {
  typedef Conv16DgradShape S;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, q4 = lane >> 4;
  const int W = a.W, Wo = a.Wo, TQ = a.TQ, RP = (Wo + 1) * 64, dyimg_bytes = S::dyimg_bytes(Wo, TQ), rowbytes = Wo * 64, segs = (rowbytes + 1023) >> 10;
  char* const stage = lds + 2 * dyimg_bytes;
  const int vb = xcd_block((int)blockIdx.x, (int)gridDim.x);
  const int nq = (a.ntiles > vb) ? (a.ntiles - 1 - vb) / (int)gridDim.x + 1 : 0;
  // the slot right of every row is zeros
  for (int i = tid; i < 2 * (TQ + 1) * 4; i += S::THREADS) *reinterpret_cast<uint4*>(lds + (i >> 2) * RP + Wo * 64 + (i & 3) * 16) = make_uint4(0u, 0u, 0u, 0u);
  bf16x8_t w[9];  // lane: result channel l16, gradient channels 8 q4 ..
#pragma unroll
  for (int s = 0; s < 9; ++s) w[s] = *reinterpret_cast<const bf16x8_t*>(a.wt + (s * S::CI + l16) * S::CO + q4 * 8);
  auto issue = [&](int q) __attribute__((always_inline)) {
    const int t = vb + q * gridDim.x, img = (int)a.dv_rb0.div((uint32_t)t), band = t - img * a.NB, oy_lo = band * TQ;
    const char* src = reinterpret_cast<const char*>(a.dy.ptr_uniform(img)) + (int64_t)oy_lo * rowbytes;
    char* dst = lds + (q & 1) * dyimg_bytes;
    for (int row = wave; row <= TQ; row += 4) {
      const bool inside = oy_lo + row < a.Ho;
#pragma unroll
      for (int sg = 0; sg < S::MAXSEG; ++sg)
        if (sg < segs) {
          const uint32_t phys = sg * 1024 + lane * 16, logi = phys ^ (((phys >> 8) & 3u) << 4);
          const char* p = inside ? src + (int64_t)row * rowbytes + logi : reinterpret_cast<const char*>(a.zpage) + lane * 16;
          if ((int)phys < rowbytes) __builtin_amdgcn_global_load_lds(GLOBAL_AS(p), LDS_AS(dst + row * RP + sg * 1024), 16, 0, LOAD_NT);
        }
    }
  };
  int stores = 0;  // this wave's stores behind the loads of the tile to come
  if (nq > 0) issue(0);
  for (int q = 0; q < nq; ++q) {
    const int t = vb + q * gridDim.x, img = (int)a.dv_rb0.div((uint32_t)t), band = t - img * a.NB;
    vm_wait_few(stores);  // the band's loads have landed
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();  // everybody's have, and the stage has been read
    if (q + 1 < nq) issue(q + 1);
    const int rows = min(2 * TQ, a.H - 2 * band * TQ);
#pragma unroll
    for (int gq = 0; gq < 2; ++gq) {
      const int qi = (wave + 4 * gq) * 16 + l16;
      const bool in_band = qi < TQ * Wo;
      const int al = in_band ? (int)a.dv_wo.div((uint32_t)qi) : 0, b = in_band ? qi - al * Wo : 0;
      const char* im = lds + (q & 1) * dyimg_bytes + al * RP;
      bf16x8_t x[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const int px = b + (p & 1);
        x[p] = *reinterpret_cast<const bf16x8_t*>(im + (p >> 1) * RP + px * 64 + ((uint32_t)(q4 ^ ((px >> 2) & 3)) << 4));
      }
      cs_f4 r[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) r[c] = cs_f4{0.f, 0.f, 0.f, 0.f};
      // class (py, px) takes tap u = py ? (dyo ? 0 : 2) : 1 from row offset dyo (even rows only from dyo = 0), same for columns
      r[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[4], x[0], r[0], 0, 0, 0);
      r[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[5], x[0], r[1], 0, 0, 0);
      r[2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[7], x[0], r[2], 0, 0, 0);
      r[3] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[8], x[0], r[3], 0, 0, 0);
      r[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[3], x[1], r[1], 0, 0, 0);
      r[3] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[6], x[1], r[3], 0, 0, 0);
      r[2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[1], x[2], r[2], 0, 0, 0);
      r[3] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[2], x[2], r[3], 0, 0, 0);
      r[3] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[0], x[3], r[3], 0, 0, 0);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int y = 2 * al + (c >> 1), xx = 2 * b + (c & 1);
        if (in_band && xx < W && y < rows) *reinterpret_cast<uint2*>(stage + (y * W + xx) * 32 + q4 * 8) = make_uint2(pack2bf(r[c][0], r[c][1]), pack2bf(r[c][2], r[c][3]));
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();  // the band is staged
    const int bi = img / a.V, vw = img - bi * a.V, nvalid = rows * W * 2;  // 16-byte pieces
    bf16_t* const out = a.dx + (int64_t)bi * a.x_stride_b + (int64_t)vw * a.x_stride_v + (int64_t)(2 * band * TQ) * W * S::CI;
    stores = 0;
    for (int c = wave * 64; c < nvalid; c += S::THREADS) {
      ++stores;
      if (c + lane < nvalid) store_stream16(out + (int64_t)(c + lane) * 8, *reinterpret_cast<const uint4*>(stage + (c + lane) * 16));
    }
  }
}
