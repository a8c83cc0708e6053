// Weight and bias gradient of the first convolution (1 or 3 input channels, 3x3 stride 2 pad 1) from a stored output
// gradient: dW[co][k] = sum over pixels dY[p][co] * patch[p][k], db[co] = sum dY[p][co] (k = 9*C0: a column of ones).
// For the networks whose layer normalisation keeps this gradient in memory (elsewhere it never leaves the chip,
// conv_dgrad_wgrad0_tile.hip.h).  The work is reading dY once (2*Cout bytes per pixel against 10 multiply-adds per
// channel): what must not pace it is the patch gather, nine 2-byte values per pixel, and index arithmetic per pixel
// (the pixel-by-pixel kernel this replaces ran at 1.1 TB/s for that reason).
//
// Bands of output rows go through an LDS ring as in conv0_tile.hip.h: the band's dY is one contiguous span, its
// 2*TR + 1 image rows another; four loader waves keep two bands in flight with LDS-writing 16-byte loads.  Four compute
// waves take 32 pixels per step (four lane groups x 8 pixels of one output row; a row's last step repeats pixel 0 with
// a zero patch): 16x16x32 MFMAs with dY^T (16 channels, transposing LDS reads) against the patches (16 columns).  A lane
// owns one patch column; its eight values are the same half of eight consecutive dwords when C0 = 1 (four two-dword
// reads and four byte permutes).  Accumulators stay in registers over all bands; a block leaves one partial
// [Cout][9*C0 + 1], summed in block order by k_reduce_batch.
// 4096 images of 60x80x16: 712 -> 157 us (0.79 GB, 5.0 TB/s).
#pragma once
#include "conv0_tile.hip.h"

struct Conv0WgradArgs {
  ImgAddr in;           // images [H][W][C0], gathered through in.idx
  const bf16_t* dy;     // [img][Ho][Wo][Cout], dense
  const bf16_t* zpage;  // 1 KiB of zeros
  float* partial;       // [gridDim.x][Cout][9*C0 + 1]
  int H, W, Ho, Wo;
  int TR, NB, ntiles;   // output rows per band, bands per image, nimg * NB
  FastDiv dv_rb;        // division by the bytes of an image row
};

template <int C0, int CO>
struct Conv0WgradShape {
  static constexpr int K0 = 9 * C0, NT = (K0 + 1 + 15) / 16, MT = (CO + 15) / 16, NBUF = 3, THREADS = 512;
  // dY behind the image rows, with room for the channels and pixels read beyond the band's end
  __host__ __device__ static int img_bytes(int W, int TR) { return (2 * TR + 1) * W * C0 * 2 + 32; }
  __host__ __device__ static int dy_bytes(int Wo, int TR) { return TR * Wo * CO * 2; }
  __host__ __device__ static int buf_bytes(int W, int Wo, int TR) { return img_bytes(W, TR) + dy_bytes(Wo, TR) + 32; }
  static int lds_bytes(int W, int Wo, int TR) {
    const int ring = NBUF * buf_bytes(W, Wo, TR) + 64, red = 4 * MT * NT * 256 * 4;
    return ring > red ? ring : red;
  }
};

template <int C0, int CO>
__global__ __launch_bounds__(512) void k_conv0_wgrad_tile(Conv0WgradArgs a) {
  typedef Conv0WgradShape<C0, CO> S;
  constexpr int K0 = S::K0, NT = S::NT, MT = S::MT, NBUF = S::NBUF;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int W = a.W, TR = a.TR, Wo = a.Wo, RB = W * C0 * 2, irows = (2 * TR + 1) * RB;
  const int dy_off = S::img_bytes(W, TR), dy_bytes = S::dy_bytes(Wo, TR), buf_bytes = S::buf_bytes(W, Wo, TR);
  const int vb = xcd_block((int)blockIdx.x, (int)gridDim.x);
  const int nq = (a.ntiles > vb) ? (a.ntiles - 1 - vb) / (int)gridDim.x + 1 : 0;
  char* const ring = lds + 32;  // the patch of column -1 starts up to 6 bytes in front of a row

  // nothing uninitialised may meet a zero patch (a NaN times zero is none): clear the ring once
  for (int i = tid; i < (NBUF * buf_bytes + 64) / 16; i += S::THREADS) reinterpret_cast<uint4*>(lds)[i] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();

  if (wave >= 4) {
    // ------------------------------------------------------------------ loaders: 1 KiB pieces in turn
    const int lw = wave - 4, n0 = (irows + 1023) >> 10, n1 = (dy_bytes + 1023) >> 10;
    const int ni = ((n0 - lw + 3) >> 2) + ((n1 - lw + 3) >> 2);
    int slot = 0;
    auto issue = [&](int q) {
      const int t = vb + q * gridDim.x, img = t / a.NB, band = t - img * a.NB;
      const int iy_lo = 2 * band * TR - 1;
      const char* isrc = reinterpret_cast<const char*>(a.in.ptr_uniform(img)) + (int64_t)iy_lo * RB;
      const char* dsrc = reinterpret_cast<const char*>(a.dy + ((int64_t)img * a.Ho + (int64_t)band * TR) * Wo * CO);
      const int dlim = min(TR, a.Ho - band * TR) * Wo * CO * 2;
      const char* zp = reinterpret_cast<const char*>(a.zpage) + lane * 16;
      char* buf = ring + slot * buf_bytes;
      slot = slot + 1 == NBUF ? 0 : slot + 1;
      for (int j = lw; j < n0; j += 4) {
        const int o = j * 1024 + lane * 16, iy = iy_lo + (int)a.dv_rb.div((uint32_t)o);
        const char* p = (iy >= 0 && iy < a.H) ? isrc + o : zp;
        if (o < irows) __builtin_amdgcn_global_load_lds(GLOBAL_AS(p), LDS_AS(buf + j * 1024), 16, 0, 0);
      }
      for (int j = lw; j < n1; j += 4) {
        const int o = j * 1024 + lane * 16;
        const char* p = o < dlim ? dsrc + o : zp;
        if (o < dy_bytes) __builtin_amdgcn_global_load_lds(GLOBAL_AS(p), LDS_AS(buf + dy_off + j * 1024), 16, 0, LOAD_NT);
      }
    };
    if (nq > 0) issue(0);
    if (nq > 1) issue(1);
    for (int q = 0; q < nq; ++q) {
      vm_wait_dyn(q + 1 < nq ? ni : 0);  // band q has landed
      __builtin_amdgcn_s_barrier();
      if (q + 2 < nq) issue(q + 2);
    }
    __syncthreads();  // the compute waves' sums are in LDS
    __syncthreads();
    return;
  }

  // -------------------------------------------------------------------- compute waves
  typedef __attribute__((ext_vector_type(4))) float f32x4_t;
  const int g = lane >> 4, r16 = lane & 15;
  f32x4_t acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[i][n] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  // this lane's patch columns: byte offset of (tap row u, tap column v, channel) from the window's column 0
  int koff[NT]; bool kone[NT], kval[NT]; uint32_t ksel[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    const int k = n * 16 + r16, kk = k < K0 ? k : 0, tap = kk / C0, ch = kk - tap * C0, u = tap / 3, v = tap - 3 * u;
    kval[n] = k < K0; kone[n] = k == K0;
    const int o = u * RB + ((v - 1) * C0 + ch) * 2;    // may be negative: one element to the left of the row
    koff[n] = C0 == 1 ? (o & ~3) : o;                  // one channel: the dword that holds it ...
    ksel[n] = (o & 2) ? 0x07060302u : 0x05040100u;     // ... and its half, of two dwords at a time
  }
  const int spr = (Wo + 31) >> 5, nstep = TR * spr;    // 32-pixel steps per row and band
  int slot = 0;
  for (int q = 0; q < nq; ++q) {
    __builtin_amdgcn_s_barrier();
    const char* buf = ring + slot * buf_bytes;
    slot = slot + 1 == NBUF ? 0 : slot + 1;
    for (int st = wave; st < nstep; st += 4) {
      const int oyl = st / spr, x0 = (st - oyl * spr) * 32 + g * 8;  // this lane group's 8 pixels
      const int nx = Wo - x0, xs = nx > 0 ? x0 : 0;                   // nx <= 0: none exist (pixel 0 with a zero patch)
      // dY^T: lane supplies 4 channels of pixel r16 / 4 (+ 4), receives channel r16 of 8 pixels
      // (pixels beyond the row's end are the next row's or the band's last: finite values that meet a zero patch)
      const int px = oyl * Wo + xs + (r16 >> 2), plast = TR * Wo - 1;
      const char* d0 = buf + dy_off + 8 * (r16 & 3);
      const char *dlo = d0 + min(px, plast) * (CO * 2), *dhi = d0 + min(px + 4, plast) * (CO * 2);
      bf16x8_t av[MT];
#pragma unroll
      for (int i = 0; i < MT; ++i) av[i] = lds_read_tr8_2(dlo + i * 32, dhi + i * 32);
      const char* ip = buf + (2 * oyl) * RB + 2 * xs * C0 * 2;
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        uint32_t w[4] = {0u, 0u, 0u, 0u};
        if constexpr (C0 == 1) {
          const uint32_t* d = reinterpret_cast<const uint32_t*>(ip + koff[n]);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int e = 2 * j < nx ? 2 * j : 0;  // stay inside the row's data for groups that reach beyond it
            w[j] = __builtin_amdgcn_perm(d[e + 1], d[e], ksel[n]);
          }
          // the window's left column of pixel 0 is outside the image
          if (r16 % 3 == 0 && xs == 0) w[0] &= 0xffff0000u;
        } else {
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int e = j < nx ? j : 0;
            uint32_t x = *reinterpret_cast<const uint16_t*>(ip + koff[n] + e * 4 * C0);
            if (j == 0 && xs == 0 && (n * 16 + r16) / C0 % 3 == 0) x = 0u;
            w[j >> 1] |= x << (16 * (j & 1));
          }
        }
        uint32_t one = 0x3F803F80u;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint32_t live = (2 * j < nx ? 0x0000ffffu : 0u) | (2 * j + 1 < nx ? 0xffff0000u : 0u);
          w[j] = (kone[n] ? one : kval[n] ? w[j] : 0u) & live;
        }
        const bf16x8_t bv = __builtin_bit_cast(bf16x8_t, make_uint4(w[0], w[1], w[2], w[3]));
#pragma unroll
        for (int i = 0; i < MT; ++i) acc[i][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[i], bv, acc[i][n], 0, 0, 0);
      }
    }
  }
  // acc[i][n][e] = dW[co = i*16 + g*4 + e][k = n*16 + r16]: the four waves' sums meet in LDS
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  float* red = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int e = 0; e < 4; ++e) red[((wave * MT + i) * NT + n) * 256 + (g * 4 + e) * 16 + r16] = acc[i][n][e];
  __syncthreads();
  float* P = a.partial + (int64_t)blockIdx.x * CO * (K0 + 1);
  for (int o = tid; o < CO * (K0 + 1); o += 256) {
    const int co = o / (K0 + 1), k = o - co * (K0 + 1), s = ((co >> 4) * NT + (k >> 4)) * 256 + (co & 15) * 16 + (k & 15);
    constexpr int WS = MT * NT * 256;
    P[o] = (red[s] + red[s + WS]) + (red[s + 2 * WS] + red[s + 3 * WS]);
  }
}
