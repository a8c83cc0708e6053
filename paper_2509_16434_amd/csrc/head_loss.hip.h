// The network's output layer (policy means and value: NH <= 32 columns), the loss, and the output
// layer's backward in one kernel.  Each of these is tiny; as separate launches (a GEMM, the loss, a
// weight-gradient GEMM with its partial sums, an input-gradient GEMM) their fixed costs dominate an
// optimiser step at small batch sizes.
//
// A block of 256 threads takes 64 samples:
//   1. the samples' last hidden activations H (64 x HID bf16) and the head weights W (NH x HID) go to LDS;
//   2. O = H W^T + b (fp32) with 32x32x16 MFMAs (waves 0 and 1, 32 samples each);
//   3. four lanes per sample, eight columns each, evaluate the loss: the gradient row dO (bf16, 32
//      columns) stays in LDS; the sums over the samples (statistics, log-std gradient, column sums of
//      dO) are taken by eight lanes per column and leave as one partial per block;
//   4. dH = dO W, masked by H > 0 (ReLU), rounded to bf16, staged and written out as full rows
//      (wave w: hidden units 32w .. 32w+31);
//   5. this block's term of dW = dO^T H (contraction over the 64 samples; both operands are row-major
//      over samples and are read with transposing LDS reads, as in k_wgrad) leaves as an fp32 partial,
//      summed afterwards in block order.
// Operand rounding is that of the separate kernels: bf16 H, W, dO and dH, fp32 accumulation.
// Bound by latency (a block is alone on its CU; its 64 samples' gathers, then one dependent chain): with one lane per
// sample and 36 block sums by butterfly in every wave it took 18.0 us for 4096 samples and 128 hidden units
// (13.4 for 256 and 64), with the columns dealt to four lanes 10.5 (8.3).
#pragma once
#include "gemm.hip.h"
#include "mem_kernels.hip.h"

struct HeadLossArgs {
  const bf16_t* h;        // [n][HID] last hidden activations (after ReLU)
  const bf16_t* w;        // [NH][HID] head weights
  const bf16_t* wt;       // [HID][32] their transpose, zero padded
  const float* bias;      // [NH]
  bf16_t* dh;             // [n][HID] gradient of h, ReLU-masked
  float* wpart;           // [gridDim.x][NH][HID]
  float* bpart;           // [gridDim.x][NH]
  float* stat_part;       // [gridDim.x][LOSS_NSTAT]
  float* dls_part;        // [gridDim.x][32] (PPO only)
  int n, NH;
};

template <int HID>
struct HeadLossShape {
  static constexpr int HPA = HID + 8;    // pitch of the copy read row-wise (16 bytes mod 256: 16 rows tile the banks)
  static constexpr int HPB = HID + 32;   // pitch of the copy read through transposing reads (64 bytes mod 256)
  static constexpr int DPA = 40, DPB = 96;
  static constexpr int OFF_HA = 0, OFF_HB = OFF_HA + 64 * HPA * 2, OFF_W = OFF_HB + 64 * HPB * 2, OFF_O = OFF_W + 32 * HPA * 2;
  static constexpr int OFF_DA = OFF_O + 64 * 33 * 4, OFF_DB = OFF_DA + 64 * DPA * 2, OFF_DH = OFF_DB + 64 * DPB * 2, OFF_RED = OFF_DH + 64 * HPA * 2;
  static constexpr int LDS_BYTES = OFF_RED + (64 * 4 + 64) * 4;
};

template <int HID, bool DISTILL>
__global__ __launch_bounds__(256) void k_head_loss(HeadLossArgs a, LossData L) {
  typedef HeadLossShape<HID> S;
  static_assert(HID % 32 == 0 && HID >= 32 && HID <= 128, "one 32-wide tile of hidden units per wave");
  constexpr int HPA = S::HPA, HPB = S::HPB, DPA = S::DPA, DPB = S::DPB, NT = HID / 32;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  bf16_t* const Ha = reinterpret_cast<bf16_t*>(lds + S::OFF_HA);
  bf16_t* const Hb = reinterpret_cast<bf16_t*>(lds + S::OFF_HB);
  bf16_t* const Ws = reinterpret_cast<bf16_t*>(lds + S::OFF_W);
  float* const Os = reinterpret_cast<float*>(lds + S::OFF_O);
  bf16_t* const Da = reinterpret_cast<bf16_t*>(lds + S::OFF_DA);
  bf16_t* const Db = reinterpret_cast<bf16_t*>(lds + S::OFF_DB);
  bf16_t* const DHs = reinterpret_cast<bf16_t*>(lds + S::OFF_DH);
  float* const stt = reinterpret_cast<float*>(lds + S::OFF_RED);  // [64][4] statistics
  float* const sgl = stt + 64 * 4;                               // sig_inv[32], ls[32]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, h = lane >> 5;
  const int s0 = blockIdx.x * 64, ns = min(64, a.n - s0);  // this block's samples

  // step 3's sample and first column of this thread; the gathers from the rollout start now: their latency passes during
  // steps 1 and 2
  const int sl = tid >> 2, c0 = (tid & 3) * 8;
  LossColumns smp = {};
  if (sl < ns) smp = loss_gather_columns(L, (int64_t)L.idx[s0 + sl], c0, !DISTILL);

  // ---- 1. H rows (zeros beyond the chunk) in both pitches, W rows (zeros beyond NH)
  constexpr int CPR = HID / 8;  // 16-byte chunks per row
  for (int c = tid; c < 64 * CPR; c += 256) {
    const int r = c / CPR, cg = c - r * CPR;
    const uint4 v = r < ns ? *reinterpret_cast<const uint4*>(a.h + (int64_t)(s0 + r) * HID + cg * 8) : make_uint4(0u, 0u, 0u, 0u);
    *reinterpret_cast<uint4*>(Ha + r * HPA + cg * 8) = v;
    *reinterpret_cast<uint4*>(Hb + r * HPB + cg * 8) = v;
  }
  for (int c = tid; c < 32 * CPR; c += 256) {
    const int r = c / CPR, cg = c - r * CPR;
    *reinterpret_cast<uint4*>(Ws + r * HPA + cg * 8) = r < a.NH ? *reinterpret_cast<const uint4*>(a.w + (int64_t)r * HID + cg * 8) : make_uint4(0u, 0u, 0u, 0u);
  }
  if (!DISTILL && tid < L.A) { sgl[32 + tid] = L.logstd[tid]; sgl[tid] = __expf(-L.logstd[tid]); }
  __syncthreads();

  // ---- 2. O[s][j] = sum_k H[s][k] W[j][k] + b[j]: wave t < 2 takes samples 32t .. 32t+31
  if (wave < 2) {
    f32x16_t acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
#pragma unroll
    for (int ks = 0; ks < HID / 16; ++ks) {
      const bf16x8_t bw = *reinterpret_cast<const bf16x8_t*>(Ws + l32 * HPA + ks * 16 + h * 8);
      const bf16x8_t ah = *reinterpret_cast<const bf16x8_t*>(Ha + (wave * 32 + l32) * HPA + ks * 16 + h * 8);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bw, ah, acc, 0, 0, 0);
    }
    // acc[g*4+q] = O[sample wave*32 + l32][column g*8 + h*4 + q]
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int j = (e >> 2) * 8 + h * 4 + (e & 3);
      Os[(wave * 32 + l32) * 33 + j] = acc[e] + (j < a.NH ? a.bias[j] : 0.f);
    }
  }
  __syncthreads();

  // ---- 3. the loss: columns c0 .. c0 + 7 of sample sl (a sample beyond the chunk has zeros everywhere)
  {
    float o[8], g[8], dls[8], st[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 8; ++j) { o[j] = Os[sl * 33 + c0 + j]; g[j] = 0.f; dls[j] = 0.f; }
    if (DISTILL) mse_loss_columns(L, smp, c0, o, g, st);
    else ppo_loss_columns(L, sgl, sgl + 32, smp, c0, o, g, st, dls);
    uint4 v = make_uint4(pack2bf(g[0], g[1]), pack2bf(g[2], g[3]), pack2bf(g[4], g[5]), pack2bf(g[6], g[7]));
    if (sl >= ns) {
      v = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
      for (int j = 0; j < 8; ++j) dls[j] = 0.f;
#pragma unroll
      for (int k = 0; k < 4; ++k) st[k] = 0.f;
    }
    // the gradient row in both pitches; the terms of the sums, the log-std gradient's in the place of the outputs just read
    *reinterpret_cast<uint4*>(Da + sl * DPA + c0) = v;
    *reinterpret_cast<uint4*>(Db + sl * DPB + c0) = v;
    if (!DISTILL) {
#pragma unroll
      for (int j = 0; j < 8; ++j) Os[sl * 33 + c0 + j] = dls[j];
    }
    if ((tid & 3) == 0) *reinterpret_cast<float4*>(stt + sl * 4) = make_float4(st[0], st[1], st[2], st[3]);
  }
  __syncthreads();
  // column sums over the samples: eight lanes per column, eight samples each, in a fixed order
  {
    const int col = tid >> 3, r0 = (tid & 7) * 8;
    float sd = 0.f, sb = 0.f, ss = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (!DISTILL) sd += Os[(r0 + i) * 33 + col];
      sb += bf2f(Da[(r0 + i) * DPA + col]);
      ss += stt[(r0 + i) * 4 + (col & 3)];
    }
#pragma unroll
    for (int off = 1; off < 8; off <<= 1) { sd += __shfl_xor(sd, off); sb += __shfl_xor(sb, off); ss += __shfl_xor(ss, off); }
    if ((tid & 7) == 0) {
      if (col < a.NH) a.bpart[(int64_t)blockIdx.x * a.NH + col] = sb;
      if (!DISTILL && col < L.A) a.dls_part[(int64_t)blockIdx.x * 32 + col] = sd;
      if (col < 4) a.stat_part[(int64_t)blockIdx.x * LOSS_NSTAT + col] = ss;
    }
  }

  // ---- 4. dH[s][n] = sum_j dO[s][j] W[j][n], hidden units 32*wave .. +31 (waves beyond HID/32 idle)
  if (wave < NT) {
    bf16x8_t wt[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) wt[ks] = *reinterpret_cast<const bf16x8_t*>(a.wt + (int64_t)(wave * 32 + l32) * HEAD_LD + ks * 16 + h * 8);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      f32x16_t acc;
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[e] = 0.f;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const bf16x8_t dv = *reinterpret_cast<const bf16x8_t*>(Da + (t * 32 + l32) * DPA + ks * 16 + h * 8);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wt[ks], dv, acc, 0, 0, 0);
      }
      // acc[g*4+q] = dH[sample t*32 + l32][unit wave*32 + g*8 + h*4 + q]; keep where the activation is positive
      const int sr = t * 32 + l32;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int nn = wave * 32 + g * 8 + h * 4;
        const uint2 hv = *reinterpret_cast<const uint2*>(Ha + sr * HPA + nn);
        auto pos = [](uint32_t m) -> uint32_t { return (((short)(m & 0xffffu) > 0) ? 0x0000ffffu : 0u) | (((short)(m >> 16) > 0) ? 0xffff0000u : 0u); };
        uint2 o;
        o.x = pack2bf(acc[g * 4], acc[g * 4 + 1]) & pos(hv.x);
        o.y = pack2bf(acc[g * 4 + 2], acc[g * 4 + 3]) & pos(hv.y);
        *reinterpret_cast<uint2*>(DHs + sr * HPA + nn) = o;
      }
    }
  }

  // ---- 5. dW[j][n] partial = sum over the block's samples of dO[s][j] H[s][n]; transposing reads as in k_wgrad
  if (wave < NT) {
    const int g4 = lane >> 4, r16 = lane & 15;
    const int srow = 8 * (g4 >> 1) + (r16 >> 2), scol = 16 * (g4 & 1) + 4 * (r16 & 3);
    f32x16_t acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const bf16x8_t av = lds_read_tr8(Db + (ks * 16 + srow) * DPB + scol, 4 * DPB);
      const bf16x8_t bv = lds_read_tr8(Hb + (ks * 16 + srow) * HPB + wave * 32 + scol, 4 * HPB);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, acc, 0, 0, 0);
    }
    // acc[g*4+q] = dW[j = g*8 + h*4 + q][n = wave*32 + l32]
    float* P = a.wpart + (int64_t)blockIdx.x * a.NH * HID;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int j = (e >> 2) * 8 + h * 4 + (e & 3);
      if (j < a.NH) P[j * HID + wave * 32 + l32] = acc[e];
    }
  }
  __syncthreads();
  // ---- dH rows leave as 16-byte segments
  for (int c = tid; c < 64 * CPR; c += 256) {
    const int r = c / CPR, cg = c - r * CPR;
    if (r < ns) *reinterpret_cast<uint4*>(a.dh + (int64_t)(s0 + r) * HID + cg * 8) = *reinterpret_cast<const uint4*>(DHs + r * HPA + cg * 8);
  }
}

// Output layer of the policy step and of ppo_forward: means and value of 32 samples per wave, and (SAMPLE) the action
// drawn from them, in one kernel; as a GEMM and a kernel behind it the two cost a launch and a round trip through the
// head-output rows (64 environments: 3.9 + 3.7 us plus the gap between them).  Bound by latency: every operand of the
// wave is requested at once, straight into registers (HID <= 128: eight 16-byte pieces of H and of W per lane), and
// the noise with them.  D = W H^T: a lane ends up with sample l32's columns g*8 + h*4 + q, the two halves' terms of
// the log-probability are added once at the end.
struct HeadActArgs {
  const bf16_t* h;        // [n][HID] last hidden activations
  const bf16_t* w;        // [NH][HID]
  const float* bias;      // [NH]
  int n, A, NH;
  const float *logstd, *noise;            // SAMPLE: [A], [n][A]
  float *o_action, *o_logp, *o_value;     // SAMPLE: the rollout slab's rows
  float *c_action, *c_logp, *c_value;     // the caller's rows, each optional: actions (SAMPLE) or means, log-probs, values
};
// A wave's operands but the hidden activations, and what follows them.  s: sample l32 of the wave (live: it exists).
template <int HID, bool SAMPLE>
struct HeadActRegs {
  static constexpr int KS = HID / 16;
  bf16x8_t bw[KS];
  float xi[16], ls[16];
  f32x16_t acc;  // starts at the bias
  __device__ __forceinline__ void load(const HeadActArgs& a, int s, bool live, int l32, int h) {
    const bf16_t* const wr = a.w + (int64_t)(l32 < a.NH ? l32 : 0) * HID + h * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) bw[ks] = *reinterpret_cast<const bf16x8_t*>(wr + ks * 16);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int j = (e >> 2) * 8 + h * 4 + (e & 3);
      acc[e] = a.bias[j < a.NH ? j : 0];
      if (SAMPLE) { const int ja = j < a.A ? j : 0; xi[e] = a.noise[(int64_t)(live ? s : 0) * a.A + ja]; ls[e] = a.logstd[ja]; }
    }
  }
  __device__ __forceinline__ void finish(const HeadActArgs& a, const bf16x8_t (&ah)[KS], int s, bool live, int h) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bw[ks], ah[ks], acc, 0, 0, 0);
    // (rows of W beyond NH repeated row 0; their columns are not used)
    float logp = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int j = (e >> 2) * 8 + h * 4 + (e & 3);
      if (j < a.A) {
        float x = acc[e];
        if (SAMPLE) {  // the arithmetic of k_act_sample
          const float mu = x, sg = expf(ls[e]), sig_inv = __expf(-ls[e]);
          x = mu + sg * xi[e];
          const float zz = (x - mu) * sig_inv;
          logp += -0.5f * zz * zz - ls[e] - 0.91893853320467274178f;
          if (live) a.o_action[(int64_t)s * a.A + j] = x;
        }
        if (live && a.c_action) a.c_action[(int64_t)s * a.A + j] = x;
      } else if (j == a.A && j < a.NH) {
        if (SAMPLE && live) a.o_value[s] = acc[e];
        if (live && a.c_value) a.c_value[s] = acc[e];
      }
    }
    if (SAMPLE) {
      const float other = __shfl_xor(logp, 32);
      const float lp = h ? other + logp : logp + other;
      if (live && h == 0) { a.o_logp[s] = lp; if (a.c_logp) a.c_logp[s] = lp; }
    }
  }
};
template <int HID, bool SAMPLE>
__global__ __launch_bounds__(64) void k_head_act(HeadActArgs a) {
  constexpr int KS = HID / 16;
  const int lane = threadIdx.x, l32 = lane & 31, h = lane >> 5, s = blockIdx.x * 32 + l32;
  const bool live = s < a.n;
  const bf16_t* const hr = a.h + (int64_t)(live ? s : 0) * HID + h * 8;
  bf16x8_t ah[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) ah[ks] = *reinterpret_cast<const bf16x8_t*>(hr + ks * 16);
  HeadActRegs<HID, SAMPLE> r;
  r.load(a, s, live, l32, h);
  r.finish(a, ah, s, live, h);
}
