// The small network (both convolutions of conv_small.hip.h, one hidden layer of 32 or 64 units) forward in one kernel, from the
// images to the hidden activations or, in the policy step, to the sampled action: there the images come from the caller and are
// stored in the rollout buffer on the way.  As separate kernels (buffer write, convolutions, hidden layer, output layer) such a
// pass is a chain of launches that each do little: 64 environments of 32x32 took 19.8 us the policy step,
// now 10.5 (1024: 20.1 and 14.8); 256 samples to the hidden layer 11.6 us in two launches, now 10.4 in one.
//
// A block of eight waves takes S samples, one after the other through the convolutions, then all of them through the hidden
// layer: its weights (a wave's slice of K, all outputs) are requested when the block starts and arrive while the
// convolutions run.  S keeps the grid within the chip's 256 CUs: more blocks would each read the weights again.  Bound by latency:
// the image, two barriers a convolution, one dependent chain of products.
//
// The sums are those of the separate kernels, bit for bit: the convolutions' own code, k_gemm_small's slices of K (as many as
// there, two accumulators in turn, added in wave order) and k_head_act's output layer.
#pragma once
#include "conv_small.hip.h"
#include "head_loss.hip.h"

struct SmallNetArgs {
  ConvSmallArgs cs;             // images (TRAIN: gathered), weights, feature rows (TRAIN), proprioception (TRAIN)
  const void* src;              // ACT: the caller's images [n][H][W0], fp32 or bf16
  const float* psrc;            // ACT: the caller's proprioception [n][P]
  bf16_t *slab, *pslab;         // ACT: where both are stored
  int W0;                       // ACT: the caller's row length
  int n, S;                     // samples, of a block
  int K, per;                   // hidden layer: depth, a wave's slice (a multiple of 16)
  const bf16_t* w;              // [HID][K]
  const float* b;
  bf16_t* hout;                 // TRAIN: [n][HID]
  HeadActArgs head;             // ACT (w, bias, NH, A, logstd, noise and the outputs)
};
struct SmallNetShape {
  static constexpr int MAXS = 4;
  static int fpitch(int K) { return K * 2 + 16; }  // bytes of a sample's features
  static int lds_bytes(const ConvSmallArgs& a, int K, int S, int HID) {
    return ConvSmallShape::block_bytes(a.W, a.Ho0, a.Ho1, a.Wo1, false) + S * fpitch(K) + 8 * S * HID * 4 + S * (HID * 2 + 16);
  }
};

// NK: k-steps of 16 in a wave's slice, at most
template <typename InT, int HID, int NK, bool ACT>
__global__ __launch_bounds__(512) void k_small_net(SmallNetArgs a) {
  constexpr int NJ = HID / 32, KS = HID / 16;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, h = lane >> 5;
  const int s0 = blockIdx.x * a.S, ns = min(a.S, a.n - s0);
  const ConvSmallArgs& cs = a.cs;
  const int wb = ConvSmallShape::block_bytes(cs.W, cs.Ho0, cs.Ho1, cs.Wo1, false), ap = ConvSmallShape::ap(cs.Wo1), ip = ConvSmallShape::ip(cs.W);
  char* const im = lds;
  char* const act = im + ConvSmallShape::img_bytes(cs.W, cs.Ho0);
  char* const feat = lds + wb;
  const int fp = a.K * 2 + 16;
  float* const red = reinterpret_cast<float*>(feat + a.S * fp);             // [wave][sample][HID]
  char* const hid = reinterpret_cast<char*>(red + 8 * a.S * HID);           // rows of HID * 2 + 16 bytes
  constexpr int HP = HID * 2 + 16;

  // This thread's first eight pixels and eight columns of the proprioception of a sample, as the caller has them: requested ahead
  // of everything else, since loads return in order.
  const int rowg = cs.W >> 3, nch = cs.H * rowg, npc = cs.P >> 3;
  struct Raw { InT px[8]; float pro[8]; uint4 stored, pstored; } raw;
  auto sample_of = [&](int b) -> int64_t { return !ACT && cs.in.idx ? cs.in.idx[b] : b; };
  auto pixels = [&](int b, int64_t smp, int i, InT (&e)[8], uint4& v) __attribute__((always_inline)) {
    if constexpr (ACT) {
      const int r = (int)cs.dvr.div((uint32_t)i), x0 = (i - r * rowg) * 8, live = a.W0 - x0;
      const InT* const p = reinterpret_cast<const InT*>(a.src) + ((int64_t)b * cs.H + r) * a.W0 + x0;
      if (live >= 8) __builtin_memcpy(e, __builtin_assume_aligned(p, sizeof(InT)), sizeof e);  // 16-byte loads at any element offset
      else {
#pragma unroll
        for (int j = 0; j < 8; ++j) e[j] = j < live ? p[j] : (InT)0;
      }
    } else
      v = *reinterpret_cast<const uint4*>(cs.in.base + smp * cs.in.stride_b + (int64_t)i * 8);
  };
  auto proprio = [&](int b, int64_t smp, int i, float (&e)[8], uint4& v) __attribute__((always_inline)) {
    if constexpr (ACT) __builtin_memcpy(e, __builtin_assume_aligned(a.psrc + (int64_t)b * cs.P + i * 8, 4), sizeof e);
    else v = *reinterpret_cast<const uint4*>(cs.proprio + smp * cs.P + i * 8);
  };
  auto fetch = [&](int b) __attribute__((always_inline)) {
    const int64_t smp = sample_of(b);
    pixels(b, smp, min(tid, nch - 1), raw.px, raw.stored);
    proprio(b, smp, min(511 - tid, npc - 1), raw.pro, raw.pstored);
  };
  fetch(s0);
  __builtin_amdgcn_sched_barrier(0);
  // the hidden layer's weights of this wave's slice
  const int kb = wave * a.per, ke = min(a.K, kb + a.per);
  const bf16x8_t zero = __builtin_bit_cast(bf16x8_t, make_uint4(0u, 0u, 0u, 0u));
  bf16x8_t wr[NK][NJ];
  auto weights = [&](int i) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int k = kb + 16 * i + h * 8;  // K is a multiple of 8: a lane's eight k exist together
      wr[i][j] = k < ke ? *reinterpret_cast<const bf16x8_t*>(a.w + (int64_t)(j * 32 + l32) * a.K + k) : zero;
    }
  };
  constexpr int NE = NK < 9 ? NK : 9;  // (the others behind the convolutions, whose weights are as many registers)
#pragma unroll
  for (int i = 0; i < NE; ++i) weights(i);
  for (int i = tid; i < wb / 16; i += 512) reinterpret_cast<uint4*>(im)[i] = make_uint4(0u, 0u, 0u, 0u);
  const int g = lane >> 4, r16 = lane & 15;
  bf16x8_t w1[3];
  int toff[3];
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    const int tap = 4 * s + g, t = tap < 9 ? tap : 0;
    w1[s] = tap < 9 ? *reinterpret_cast<const bf16x8_t*>(cs.w1 + r16 * 72 + tap * 8) : zero;
    toff[s] = ((t / 3) * ap + t % 3) * 16;
  }
  const float4 b1 = *reinterpret_cast<const float4*>(cs.b1 + g * 4);
  CsW0 w0;
  cs_weights0(cs, w0);
  const int n1 = cs.Ho1 * cs.Wo1, flat = n1 * 16;
  __syncthreads();
  for (int s = 0; s < ns; ++s) {
    const int b = s0 + s;
    // ---- the image's rows and the proprioception into LDS (ACT: rounded, and into the buffer)
    auto put_pixels = [&](int i, const InT (&e)[8], uint4 v) __attribute__((always_inline)) {
      const int r = (int)cs.dvr.div((uint32_t)i), c = i - r * rowg;
      if constexpr (ACT) {
        uint32_t o[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if constexpr (sizeof(InT) == 4) o[q] = pack2bf((float)e[2 * q], (float)e[2 * q + 1]);
          else o[q] = (uint32_t)e[2 * q] | (uint32_t)e[2 * q + 1] << 16;
        }
        v = make_uint4(o[0], o[1], o[2], o[3]);
        *reinterpret_cast<uint4*>(a.slab + (int64_t)b * cs.in.stride_b + (int64_t)i * 8) = v;
      }
      *reinterpret_cast<uint4*>(im + (r + 1) * ip + 16 + c * 16) = v;
    };
    auto put_proprio = [&](int i, const float (&e)[8], uint4 v) __attribute__((always_inline)) {
      if constexpr (ACT) {
        v = make_uint4(pack2bf(e[0], e[1]), pack2bf(e[2], e[3]), pack2bf(e[4], e[5]), pack2bf(e[6], e[7]));
        *reinterpret_cast<uint4*>(a.pslab + (int64_t)b * cs.P + i * 8) = v;
      } else
        *reinterpret_cast<uint4*>(cs.feat + (int64_t)b * cs.feat_ld + flat + i * 8) = v;
      *reinterpret_cast<uint4*>(feat + s * fp + flat * 2 + i * 16) = v;
    };
    if (tid < nch) put_pixels(tid, raw.px, raw.stored);
    if (511 - tid < npc) put_proprio(511 - tid, raw.pro, raw.pstored);
    const int64_t smp = sample_of(b);
    for (int i = tid + 512; i < nch; i += 512) {
      InT e[8]; uint4 v = make_uint4(0u, 0u, 0u, 0u);
      pixels(b, smp, i, e, v);
      put_pixels(i, e, v);
    }
    for (int i = 1023 - tid; i < npc; i += 512) {
      float e[8]; uint4 v = make_uint4(0u, 0u, 0u, 0u);
      proprio(b, smp, i, e, v);
      put_proprio(i, e, v);
    }
    if (s + 1 < ns) fetch(b + 1);
    __syncthreads();
    cs_conv0<512>(cs, im, act, w0, tid);
    __syncthreads();
    for (int q = wave * 16; q < n1; q += 128) {
      const int p = q + r16, pc = p < n1 ? p : 0, y = (int)cs.dv1.div((uint32_t)pc), x = pc - y * cs.Wo1;
      const char* wp = act + (2 * y * ap + 2 * x) * 16;
      cs_f4 acc = {b1.x, b1.y, b1.z, b1.w};
#pragma unroll
      for (int t = 0; t < 3; ++t) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1[t], *reinterpret_cast<const bf16x8_t*>(wp + toff[t]), acc, 0, 0, 0);
      const uint2 o = make_uint2(relu_pack2bf(acc[0], acc[1]), relu_pack2bf(acc[2], acc[3]));
      if (p < n1) {
        *reinterpret_cast<uint2*>(feat + s * fp + (p * 16 + g * 4) * 2) = o;
        if (!ACT) *reinterpret_cast<uint2*>(cs.feat + (int64_t)b * cs.feat_ld + p * 16 + g * 4) = o;
      }
    }
    // (the next sample's image may land now: the first convolution's reads lie behind a barrier; its output is written behind another)
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = NE; i < NK; ++i) weights(i);
  __syncthreads();
  // ---- hidden layer: this wave's slice of K; column l32 of the product is sample l32 (those beyond the block repeat the first)
  {
    f32x16_t acc[NJ][2];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) { acc[j][0][e] = 0.f; acc[j][1][e] = 0.f; }
    const char* const fr = feat + (l32 < ns ? l32 : 0) * fp + h * 16;
#pragma unroll
    for (int i = 0; i < NK; ++i) {
      const int k = kb + 16 * i;
      const bf16x8_t f = k + h * 8 < ke ? *reinterpret_cast<const bf16x8_t*>(fr + k * 2) : zero;
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[j][i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wr[i][j], f, acc[j][i & 1], 0, 0, 0);
    }
    if (l32 < ns) {
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<float4*>(red + (wave * a.S + l32) * HID + j * 32 + q * 8 + h * 4) =
              make_float4(acc[j][0][q * 4] + acc[j][1][q * 4], acc[j][0][q * 4 + 1] + acc[j][1][q * 4 + 1], acc[j][0][q * 4 + 2] + acc[j][1][q * 4 + 2], acc[j][0][q * 4 + 3] + acc[j][1][q * 4 + 3]);
    }
  }
  // (ACT) the output layer's operands of wave 0
  const int s = s0 + l32;
  const bool live = ACT && l32 < ns;
  HeadActRegs<HID, ACT> hr;
  if (ACT && wave == 0) hr.load(a.head, s, live, l32, h);
  __syncthreads();
  for (int i = tid; i < ns * (HID / 4); i += 512) {
    const int r = i / (HID / 4), c = (i - r * (HID / 4)) * 4;
    float4 v = *reinterpret_cast<const float4*>(red + r * HID + c);
#pragma unroll
    for (int w = 1; w < 8; ++w) { const float4 x = *reinterpret_cast<const float4*>(red + (w * a.S + r) * HID + c); v.x += x.x; v.y += x.y; v.z += x.z; v.w += x.w; }
    const float4 bb = *reinterpret_cast<const float4*>(a.b + c);
    const uint2 o = make_uint2(pack2bf(fmaxf(v.x + bb.x, 0.f), fmaxf(v.y + bb.y, 0.f)), pack2bf(fmaxf(v.z + bb.z, 0.f), fmaxf(v.w + bb.w, 0.f)));
    if constexpr (ACT) *reinterpret_cast<uint2*>(hid + r * HP + c * 2) = o;
    else *reinterpret_cast<uint2*>(a.hout + (int64_t)(s0 + r) * HID + c) = o;
  }
  if constexpr (ACT) {
    __syncthreads();
    if (wave == 0) {
      bf16x8_t ah[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) ah[ks] = *reinterpret_cast<const bf16x8_t*>(hid + (live ? l32 : 0) * HP + ks * 32 + h * 16);
      hr.finish(a.head, ah, s, live, h);
    }
  }
}
