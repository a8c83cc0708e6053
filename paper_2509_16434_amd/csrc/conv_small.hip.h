// Both convolutions of a small network (one-channel images -> 8 -> 16 channels, 3x3 stride 2 pad 1) in one kernel per
// direction.  The layers are so thin (72 and 1152 multiply-adds per output pixel) that as separate kernels they cost
// their launches at small batches (three dependent ones forward, four backward, 5-10 us each) and the first layer's
// activation's way through memory at large ones.  A block takes one image at a time from start to end in LDS, its four
// waves sharing each phase's pixels (a wave per image leaves most of the chip idle at small batches, and at 64x64 the LDS
// of a CU holds four images, one wave per SIMD) and the next image's loads in flight: the image (rows behind 16 bytes of
// zeros), the first layer's output (16 bytes per pixel, one zero slot around), backward also the second layer's gradient
// (32 bytes per pixel).  The backward pass recomputes the
// first layer's output instead of reading it; gradients accumulate in registers over all images of a block.
//
// First layer: lane = pixel, 72 fp32 multiply-adds with the weights in registers (K = 9 is too thin for the
// matrix cores).  Second layer: 16x16x32 MFMAs, four taps of eight channels per step, so that a lane's operand is one
// 16-byte LDS read.  Its weight gradient contracts over pixels (both operands through transposing LDS reads; the tenth
// tap reads ones: the bias column).  Its input gradient works on quads (2x2 pixels of the first layer): rows 0-7 / 8-15
// of the product are the even / odd column's eight channels, k runs over the two gradient pixels a quad row touches.
// The gradient then meets the image patch of its pixel in fp32 registers.
// Against one kernel per layer: 256 images of 32x32 forward 15 -> 6.5 us, backward 22 -> 9.4; 16384 images 91 -> 35 and
// 222 -> 61 us (0.62 of the vector units' issue slots); 8000 images of 64x64 133 -> 53 and 403 -> 101 us.
#pragma once
#include "conv_tile.hip.h"

struct ConvSmallArgs {
  ImgAddr in;              // images [H][W], gathered through in.idx; W a multiple of 8
  const bf16_t *w0, *w1;   // [8][9], [16][72] (k = tap*8 + ci)
  const bf16_t* w1t;       // [9][8][16]
  const float *b0, *b1;
  bf16_t* feat;            // forward: rows [n][feat_ld], view v's output at v*flat
  const bf16_t* dfeat;     // backward: gradient rows of the same form, masked by the second layer's ReLU
  int64_t feat_ld;
  int V, flat, nimg;
  int H, W, Ho0, Wo0, Ho1, Wo1;
  FastDiv dv0, dv1, dvr;   // division by Wo0, Wo1, W / 8
  const bf16_t* proprio;   // forward: columns [V*flat, V*flat + P) of the feature rows
  int P;
  float *part1, *bpart1, *part0;  // backward: [gridDim.x][16][72], [gridDim.x][16], [gridDim.x][8][10]
};

struct ConvSmallShape {
  __host__ __device__ static int ip(int W) { return 16 + W * 2; }                       // image row pitch
  __host__ __device__ static int img_bytes(int W, int Ho0) { return (2 * Ho0 + 1) * ip(W); }
  __host__ __device__ static int ap(int Wo1) { return 2 * Wo1 + 1; }                    // slots per row of the first layer's output
  __host__ __device__ static int act_bytes(int Ho1, int Wo1) { return (2 * Ho1 + 1) * ap(Wo1) * 16; }
  __host__ __device__ static int dy_bytes(int Ho1, int Wo1) { return (Ho1 + 1) * (Wo1 + 1) * 32; }
  __host__ __device__ static int block_bytes(int W, int Ho0, int Ho1, int Wo1, bool bwd) {
    return img_bytes(W, Ho0) + act_bytes(Ho1, Wo1) + (bwd ? dy_bytes(Ho1, Wo1) + 16 : 0);
  }
  static constexpr int CHUNKS = 5;  // the kernels' CH is 1, 2 or 5
  // two blocks per CU, so that one's barriers and latencies overlap the other's arithmetic
  static bool covers(int H, int W, int Ho0, int Ho1, int Wo1) {
    return block_bytes(W, Ho0, Ho1, Wo1, true) <= 80 * 1024 && H * (W / 8) <= CHUNKS * 256 && Ho1 * Wo1 * 2 <= CHUNKS * 256;
  }
  static constexpr int RED = 16 * 80 + 80;  // floats one wave leaves for the block's sums (backward)
};

// A block's next image (and gradient) on its way in registers while the current one is worked on: CH 16-byte pieces per
// thread (ConvSmallShape::covers keeps images and gradients within CHUNKS).
struct CsRow {  // image number img of the minibatch
  int b, v;
  int64_t s;    // its sample in the buffer
};
__device__ __forceinline__ CsRow cs_row(const ConvSmallArgs& a, int img) {
  CsRow r;
  const int i = img < a.nimg ? img : 0;
  r.b = i / a.V; r.v = i - r.b * a.V;
  typedef const __attribute__((address_space(4))) int32_t* cidx_t;  // scalar load: waits for none of the vector loads in flight
  r.s = a.in.idx ? reinterpret_cast<cidx_t>(reinterpret_cast<uintptr_t>(a.in.idx))[__builtin_amdgcn_readfirstlane(r.b)] : r.b;
  return r;
}
template <int CH>
__device__ __forceinline__ void cs_fetch(const bf16_t* src, int n, int tid, uint4 (&q)[CH]) {
#pragma unroll
  for (int j = 0; j < CH; ++j)  // without a branch: a conditional load is waited for at once
    q[j] = *reinterpret_cast<const uint4*>(src + (int64_t)min(tid + j * 256, n - 1) * 8);
}
// the image's rows into LDS (the zeros in front of each row, above and below stay)
template <int CH>
__device__ __forceinline__ void cs_put_image(const ConvSmallArgs& a, char* im, int tid, const uint4 (&q)[CH]) {
  const int n = a.H * (a.W >> 3), ip = ConvSmallShape::ip(a.W);
#pragma unroll
  for (int j = 0; j < CH; ++j) {
    const int i = tid + j * 256;
    if (i < n) { const int r = (int)a.dvr.div((uint32_t)i), c = i - r * (a.W >> 3); *reinterpret_cast<uint4*>(im + (r + 1) * ip + 16 + c * 16) = q[j]; }
  }
}
// the nine window values of first-layer pixel (y, x)
__device__ __forceinline__ void cs_window(const char* im, int ip, int y, int x, float (&v)[9]) {
  const char* p = im + 2 * y * ip + 16 + 4 * x;
#pragma unroll
  for (int u = 0; u < 3; ++u) {
    const uint32_t d0 = *reinterpret_cast<const uint32_t*>(p + u * ip - 4), d1 = *reinterpret_cast<const uint32_t*>(p + u * ip);
    v[3 * u] = __uint_as_float(d0 & 0xffff0000u); v[3 * u + 1] = __uint_as_float(d1 << 16); v[3 * u + 2] = __uint_as_float(d1 & 0xffff0000u);
  }
}
// weights of the first layer, the same in every lane.  In vector registers: 80 do not fit the scalar ones, and unpacking
// bf16 pairs there costs a lone wave two more issue slots per multiply-add.
struct CsW0 { float w[8][9], b[8]; };
__device__ __forceinline__ void cs_weights0(const ConvSmallArgs& a, CsW0& q) {
  typedef const __attribute__((address_space(4))) uint32_t* cptr_t;
  const cptr_t wp = reinterpret_cast<cptr_t>(reinterpret_cast<uintptr_t>(a.w0)), bp = reinterpret_cast<cptr_t>(reinterpret_cast<uintptr_t>(a.b0));
  uint32_t w[36], b[8];
#pragma unroll
  for (int i = 0; i < 36; ++i) w[i] = wp[i];
#pragma unroll
  for (int c = 0; c < 8; ++c) b[c] = bp[c];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    q.b[c] = __uint_as_float(b[c]);
    asm volatile("" : "+v"(q.b[c]));
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      const int i = c * 9 + k;
      q.w[c][k] = __uint_as_float(i & 1 ? w[i >> 1] & 0xffff0000u : w[i >> 1] << 16);
      asm volatile("" : "+v"(q.w[c][k]));
    }
  }
}
// first layer of the image in `im` into `act`, by NT threads
template <int NT = 256>
__device__ __forceinline__ void cs_conv0(const ConvSmallArgs& a, const char* im, char* act, const CsW0& q, int tid) {
  const int ip = ConvSmallShape::ip(a.W), ap = ConvSmallShape::ap(a.Wo1), n = a.Ho0 * a.Wo0;
  for (int p = tid; p < n; p += NT) {
    const int y = (int)a.dv0.div((uint32_t)p), x = p - y * a.Wo0;
    float v[9];
    cs_window(im, ip, y, x, v);
    float o[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      o[c] = q.b[c];
#pragma unroll
      for (int k = 0; k < 9; ++k) o[c] = fmaf(v[k], q.w[c][k], o[c]);
    }
    *reinterpret_cast<uint4*>(act + ((y + 1) * ap + x + 1) * 16) =
        make_uint4(relu_pack2bf(o[0], o[1]), relu_pack2bf(o[2], o[3]), relu_pack2bf(o[4], o[5]), relu_pack2bf(o[6], o[7]));
  }
}
typedef __attribute__((ext_vector_type(4))) float cs_f4;
template <int CTRL>
__device__ __forceinline__ float cs_dpp(float x) { return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true)); }

template <int CH>
__global__ __launch_bounds__(256) void k_conv_small_fwd(ConvSmallArgs a) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nch = a.H * (a.W >> 3);
  uint4 qi[CH];
  CsRow cur = cs_row(a, blockIdx.x), nxt = cs_row(a, blockIdx.x + gridDim.x);
  const int pch = min(tid, (a.P >> 3) - 1) * 8;  // the proprioception's first 2048 columns travel the same way
  uint4 qp;
  auto fetch = [&](const CsRow& r) {
    cs_fetch(a.in.base + r.s * a.in.stride_b + r.v * a.in.stride_v, nch, tid, qi);
    qp = *reinterpret_cast<const uint4*>(a.proprio + r.s * a.P + pch);
  };
  fetch(cur);
  const int wb = ConvSmallShape::block_bytes(a.W, a.Ho0, a.Ho1, a.Wo1, false), ap = ConvSmallShape::ap(a.Wo1);
  char* const im = lds;
  char* const act = im + ConvSmallShape::img_bytes(a.W, a.Ho0);
  for (int i = tid; i < wb / 16; i += 256) reinterpret_cast<uint4*>(im)[i] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  CsW0 w0;
  cs_weights0(a, w0);
  const int g = lane >> 4, r16 = lane & 15;
  bf16x8_t w1[3];
  int toff[3];
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    const int tap = 4 * s + g, t = tap < 9 ? tap : 0;
    w1[s] = tap < 9 ? *reinterpret_cast<const bf16x8_t*>(a.w1 + r16 * 72 + tap * 8) : __builtin_bit_cast(bf16x8_t, make_uint4(0u, 0u, 0u, 0u));
    toff[s] = ((t / 3) * ap + t % 3) * 16;
  }
  const float4 b1 = *reinterpret_cast<const float4*>(a.b1 + g * 4);
  const int n1 = a.Ho1 * a.Wo1;
  for (int img = blockIdx.x; img < a.nimg; img += gridDim.x) {
    bf16_t* const out = a.feat + (int64_t)cur.b * a.feat_ld + (int64_t)cur.v * a.flat;
    if (cur.v == 0) {
      bf16_t* const po = a.feat + (int64_t)cur.b * a.feat_ld + a.V * a.flat;
      if (tid < a.P >> 3) *reinterpret_cast<uint4*>(po + pch) = qp;
      for (int j = 256 + tid; j < a.P >> 3; j += 256) reinterpret_cast<uint4*>(po)[j] = reinterpret_cast<const uint4*>(a.proprio + cur.s * a.P)[j];
    }
    cs_put_image(a, im, tid, qi);
    __syncthreads();
    cur = nxt;
    if (img + gridDim.x < a.nimg) fetch(cur);
    nxt = cs_row(a, img + 2 * gridDim.x);
    cs_conv0<>(a, im, act, w0, tid);
    __syncthreads();
    for (int q = wave * 16; q < n1; q += 64) {
      const int p = q + r16, pc = p < n1 ? p : 0, y = (int)a.dv1.div((uint32_t)pc), x = pc - y * a.Wo1;
      const char* wp = act + (2 * y * ap + 2 * x) * 16;
      cs_f4 acc = {b1.x, b1.y, b1.z, b1.w};
#pragma unroll
      for (int s = 0; s < 3; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1[s], *reinterpret_cast<const bf16x8_t*>(wp + toff[s]), acc, 0, 0, 0);
      if (p < n1) *reinterpret_cast<uint2*>(out + p * 16 + g * 4) = make_uint2(relu_pack2bf(acc[0], acc[1]), relu_pack2bf(acc[2], acc[3]));
    }
    __syncthreads();
  }
}

template <int CH>
__global__ __launch_bounds__(256) void k_conv_small_bwd(ConvSmallArgs a) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n1 = a.Ho1 * a.Wo1;
  const int nch = a.H * (a.W >> 3);
  uint4 qi[CH], qd[CH];
  CsRow nxt = cs_row(a, blockIdx.x);
  auto fetch = [&](const CsRow& r) {
    cs_fetch(a.in.base + r.s * a.in.stride_b + r.v * a.in.stride_v, nch, tid, qi);
    cs_fetch(a.dfeat + (int64_t)r.b * a.feat_ld + (int64_t)r.v * a.flat, n1 * 2, tid, qd);
  };
  fetch(nxt);
  nxt = cs_row(a, blockIdx.x + gridDim.x);
  const int wb = ConvSmallShape::block_bytes(a.W, a.Ho0, a.Ho1, a.Wo1, true), ip = ConvSmallShape::ip(a.W), ap = ConvSmallShape::ap(a.Wo1), dp = a.Wo1 + 1;
  char* const im = lds;
  char* const act = im + ConvSmallShape::img_bytes(a.W, a.Ho0);
  char* const dy = act + ConvSmallShape::act_bytes(a.Ho1, a.Wo1);
  char* const ones = dy + ConvSmallShape::dy_bytes(a.Ho1, a.Wo1);
  for (int i = tid; i < wb / 16; i += 256) reinterpret_cast<uint4*>(im)[i] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  if (tid < 4) reinterpret_cast<uint32_t*>(ones)[tid] = 0x3F803F80u;
  CsW0 w0;
  cs_weights0(a, w0);
  const int g = lane >> 4, r16 = lane & 15;
  // operands of the quad product: row r16 = column parity * 8 + ci, k = gradient pixel (g >> 1) * 16 + co half (g & 1) * 8
  bf16x8_t wq[3];
  {
    const int ci = r16 & 7, odd = r16 >> 3, src = g >> 1, half = g & 1;
    auto tap = [&](int u) {  // tap row u; columns: even pixel v = 1 from src 0; odd pixel v = 2 from src 0, v = 0 from src 1
      const int v = odd ? (src ? 0 : 2) : 1;
      return (odd || !src) ? *reinterpret_cast<const bf16x8_t*>(a.w1t + ((u * 3 + v) * 8 + ci) * 16 + half * 8) : __builtin_bit_cast(bf16x8_t, make_uint4(0u, 0u, 0u, 0u));
    };
    wq[0] = tap(1); wq[1] = tap(2); wq[2] = tap(0);  // even rows from row a; odd rows from rows a and a + 1
  }
  cs_f4 acc1[5];
#pragma unroll
  for (int t = 0; t < 5; ++t) acc1[t] = cs_f4{0.f, 0.f, 0.f, 0.f};
  float acc0[4][10];
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int k = 0; k < 10; ++k) acc0[e][k] = 0.f;
  // second layer's window columns of the weight-gradient product: tap 2t + (r16 & 3) / 2, channels (r16 & 1) * 4 ..
  int toff[5];
#pragma unroll
  for (int t = 0; t < 5; ++t) {
    const int tap = 2 * t + ((r16 & 3) >> 1);
    toff[t] = tap < 9 ? ((tap / 3) * ap + tap % 3) * 16 + (r16 & 1) * 8 : -1;
  }
  for (int img = blockIdx.x; img < a.nimg; img += gridDim.x) {
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      const int i = tid + j * 256, p = i >> 1, y = (int)a.dv1.div((uint32_t)p), x = p - y * a.Wo1;
      if (i < n1 * 2) *reinterpret_cast<uint4*>(dy + (y * dp + x) * 32 + (i & 1) * 16) = qd[j];
    }
    cs_put_image(a, im, tid, qi);
    __syncthreads();
    if (img + gridDim.x < a.nimg) fetch(nxt);
    nxt = cs_row(a, img + 2 * gridDim.x);
    cs_conv0<>(a, im, act, w0, tid);
    __syncthreads();
    // dW1[co][tap*8 + ci] += sum over pixels dY[p][co] act[window(p)][ci], 32 pixels per step
    for (int q = (3 - wave) * 32; q < n1; q += 128) {
      const char *dsrc[2], *wsrc[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int p = q + g * 8 + (r16 >> 2) + 4 * h, pc = p < n1 ? p : 0, y = (int)a.dv1.div((uint32_t)pc), x = pc - y * a.Wo1;
        dsrc[h] = dy + (p < n1 ? (y * dp + x) * 32 : a.Wo1 * 32) + (r16 & 3) * 8;  // pixels beyond the image: a zero slot
        wsrc[h] = act + (2 * y * ap + 2 * x) * 16;
      }
      const bf16x8_t av = lds_read_tr8_2(dsrc[0], dsrc[1]);
#pragma unroll
      for (int t = 0; t < 5; ++t) {
        const char* w0p = toff[t] >= 0 ? wsrc[0] + toff[t] : ones;
        const char* w1p = toff[t] >= 0 ? wsrc[1] + toff[t] : ones;
        acc1[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, lds_read_tr8_2(w0p, w1p), acc1[t], 0, 0, 0);
      }
    }
    // gradient of the first layer's output, quad by quad, and its product with the image patches
    for (int q = wave * 16; q < n1; q += 64) {
      const int p = q + r16, pc = p < n1 ? p : 0, y = (int)a.dv1.div((uint32_t)pc), x = pc - y * a.Wo1;
      const char* d = dy + (y * dp + x + (g >> 1)) * 32 + (g & 1) * 16;
      const bf16x8_t x0 = *reinterpret_cast<const bf16x8_t*>(d), x1 = *reinterpret_cast<const bf16x8_t*>(d + dp * 32);
      cs_f4 r[2];
      r[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wq[0], x0, cs_f4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
      r[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wq[1], x0, cs_f4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
      r[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wq[2], x1, r[1], 0, 0, 0);
      // this lane: pixel (2y + h, 2x + (g >> 1)), channels (g & 1) * 4 ..
      const int X = 2 * x + (g >> 1);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int Y = 2 * y + h;
        const bool ok = p < n1 && X < a.Wo0 && Y < a.Ho0;
        const uint2 m = *reinterpret_cast<const uint2*>(act + ((Y + 1) * ap + X + 1) * 16 + (g & 1) * 8);
        const uint32_t mk[4] = {m.x << 16, m.x & 0xffff0000u, m.y << 16, m.y & 0xffff0000u};
        float v9[9];
        cs_window(im, ip, ok ? Y : 0, ok ? X : 0, v9);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float dx = (ok && __uint_as_float(mk[e]) > 0.f) ? r[h][e] : 0.f;
#pragma unroll
          for (int k = 0; k < 9; ++k) acc0[e][k] = fmaf(dx, v9[k], acc0[e][k]);
          acc0[e][9] += dx;
        }
      }
    }
    __syncthreads();
  }
  // sums over the lanes that share four channels (every lane bit but bit 4), then over the waves in LDS
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int k = 0; k < 10; ++k) {
      float s = acc0[e][k];
      s += cs_dpp<0xB1>(s); s += cs_dpp<0x4E>(s); s += cs_dpp<0x141>(s); s += cs_dpp<0x140>(s);  // lanes xor 1, xor 2, then mirrored in 8 and in 16
      s += __shfl_xor(s, 32);
      acc0[e][k] = s;
    }
  __syncthreads();
  float* const red = reinterpret_cast<float*>(lds) + wave * ConvSmallShape::RED;
#pragma unroll
  for (int t = 0; t < 5; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) red[(g * 4 + e) * 80 + t * 16 + r16] = acc1[t][e];  // [co][tap*8 + ci], columns 72.. : bias
  if ((lane & 47) == 0) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int k = 0; k < 10; ++k) red[1280 + (g * 4 + e) * 10 + k] = acc0[e][k];  // lanes 0 and 16: channels 0-3, 4-7
  }
  __syncthreads();
  const float* const R = reinterpret_cast<const float*>(lds);
  auto sum = [&](int i) { float s = R[i]; for (int w = 1; w < 4; ++w) s += R[w * ConvSmallShape::RED + i]; return s; };
  for (int i = tid; i < 16 * 72; i += 256) { const int co = i / 72, k = i - co * 72; a.part1[(int64_t)blockIdx.x * 1152 + i] = sum(co * 80 + k); }
  for (int i = tid; i < 16; i += 256) a.bpart1[(int64_t)blockIdx.x * 16 + i] = sum(i * 80 + 72);
  for (int i = tid; i < 80; i += 256) a.part0[(int64_t)blockIdx.x * 80 + i] = sum(1280 + i);
}
