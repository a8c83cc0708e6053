// 3x3 stride-2 pad-1 convolution forward for 16, 32 or 64 input channels, organised around what is
// scarce on the CU for this shape: bytes in flight per CU and vector-ALU issue slots, not MFMA
// cycles.
//
//  * Persistent blocks walk over tiles = (image, band of TR output rows).  The band's input rows
//    (2*TR+1 of them, one contiguous span of the channel-last image) are copied as they are into
//    an LDS image; the im2col gather happens at LDS-read time, where a tap is a constant byte
//    offset from the lane's window corner.  Every input byte crosses the memory path once per block.
//  * The copy is done by four extra waves with loads that write LDS directly (global_load_lds_dwordx4,
//    lane l's 16 bytes land at the instruction's LDS base + 16*l), into a ring of nbuf images
//    (three for the large layers, as many as fit up to MAXBUF for small ones, whose bands are too few bytes to
//    cover the memory latency two at a time): nbuf - 1 bands are in flight while one is computed.  (One wave alone sustains only about one such
//    load per 190 cycles.)  A loader's own vmcnt counts only these loads, so "band q has landed" is an exact wait; one barrier per tile hands the image over and
//    returns the ring slot consumed one tile earlier.
//  * Each image row has a zero pixel to its left and right (written once), rows outside the image
//    are copied from a page of zeros: the padding needs no test at read time.
//  * Pixels are stored unpadded; the 16-byte chunks of a pixel are permuted by its slot index
//    (chunk ^ f(slot)), applied by the loader through the global address, so that the stride-2
//    operand reads spread over the banks (two lanes per bank group instead of eight or sixteen).
//  * A compute wave keeps its slice of the weight matrix (9*CIN deep, 64 or 32 columns: 144
//    registers) in registers for the whole kernel, and its lanes' pixel -> LDS offset is the same
//    for every tile.
//  * Each compute wave stages its 32 output pixels in a private LDS strip and writes them as
//    16-byte row segments; a band's outputs are one contiguous span of the output image.
//  * Rows too long for that (COLS): a tile is TR rows of TC output COLUMNS.  Its input is 2*TR+1 rows of 2*TC+1 pixels,
//    slot 0 being the pixel left of the tile (or padding); the rows lie back to back in LDS and are copied in 1 KiB
//    pieces that run on across row ends, every lane looking up its own source (row pitch of the image, zeros outside
//    it).  Bound by HBM like the narrow form: 120 of 128 pixels used at 80-pixel result rows in two parts, 1.18 times
//    the band's bytes loaded (a whole row of 80 would use 80 of 128 and load 1.5 times).  Measured on 8400 images of
//    240x320, against the implicit-GEMM kernels such rows took before: second and third layer together forward
//    5.74 -> 4.25 ms (5.0 TB/s of algorithmic bytes), weight gradient 6.94 -> 3.83 ms (5.6 TB/s); and with the forward's
//    sign bits the third and fourth layer's input gradient takes the LDS-image kernels too, 4.17 -> 3.09 ms.
#pragma once
#include "conv0_rows.hip.h"

struct ConvTileArgs {
  ImgAddr in;                 // input images [H][W][CIN], dense
  bf16_t* out;                // output images [Ho][Wo][Cout] at out + b*out_stride_b + v*out_stride_v
  int64_t out_stride_b, out_stride_v;
  const bf16_t* w;            // [Cout][9*CIN], k = (u*3+v)*CIN + ci
  const float* bias;          // [Cout]
  const bf16_t* zpage;        // 1 KiB of zeros
  uint32_t* bits;             // optional: one bit per output element (stored value > 0), word w of pixel p of image i at
                              // bits[(i*Ho*Wo + p) * ceil(Cout/32) + w]; read by the transposed convolution as ReLU mask
  int V, H, W, Ho, Wo, Cout;
  int TR, NB, ntiles;         // output rows per band, bands per image, nimg * NB
  int nbuf;                   // ring images (3 .. MAXBUF)
  FastDiv dv_nb, dv_np;       // division by NB, NP
  int TC, NP;                 // COLS: output columns per tile, tiles side by side (ntiles = nimg * NB * NP); else TC = Wo, NP = 1
  // C0 > 0: the input is the first layer's output, made from the images in src0; every block also copies its share of the n0
  // samples' proprioception (P values, a multiple of 8, gathered like the images) into their feature rows
  Conv0Src src0;
  Stack stk;                  // STACK: the batch as one tall image
  int n0, P;
  const bf16_t* proprio;
  bf16_t* feat;               // first column that receives it
  int64_t feat_ld;
};

template <int CIN, int WIDE = 0>
struct ConvTileShape {
  static_assert(!WIDE || CIN == 64, "the wide form is for 64 input channels");
  static constexpr int NW = (CIN == 32) ? 64 : 32;   // output columns per wave (18432 weights per wave)
  // WIDE: the four waves stand side by side (128 columns) and each takes both 32-pixel halves of the band, so that a
  // layer with more than 64 output channels loads its input once instead of once per 64 columns
  static constexpr int WGM = WIDE ? 1 : (CIN == 64) ? 2 : 4, WGN = 4 / WGM, TM = WIDE || CIN == 16 ? 2 : 1;
  static constexpr int BM = WGM * TM * 32, BN = WGN * NW;  // 128 x 64, 64 x 64 or 64 x 128; 256 x 32
  static constexpr int PIX = CIN * 2;                 // bytes per pixel
  static constexpr int MAXSEG = 6;                    // 1 KiB load instructions per image row
  static constexpr int MAXBUF = 6;
  static constexpr int SP = NW + 8;                   // staging pitch (elements)
  static constexpr int ZERO_BYTES = 3 * PIX;          // STACK
  static constexpr int STAGE_BYTES = 4 * 32 * SP * 2;
  static constexpr int THREADS = 512;                 // four compute waves + four loader waves
  static constexpr int MAXLD = 13;                    // COLS: 1 KiB loads per loader wave and tile
  static int image_bytes(int slots, int TR) { return (2 * TR + 1) * slots * PIX; }  // slots: W + 2, or 2 * TC + 1
  static int lds_bytes(int slots, int TR, int nbuf) { return nbuf * image_bytes(slots, TR) + STAGE_BYTES + BN * 4; }
};

// The loads of a tile of columns (COLS): piece j of 1 KiB belongs to loader wave j % 4.  Lane -> source is the same for
// every tile but for the image's edges: byte offset from the pixel (2*row0 - 1, 2*col0) of the image, and the row and slot.
template <int MAXLD>
struct ColsLoads {
  int goff[MAXLD];
  uint32_t rs[MAXLD];  // row | slot << 8, or ~0: nothing to load
  template <class SWZ>
  __device__ __forceinline__ void init(int lw, int lane, int image_bytes, int rp, int pix, int rowbytes, SWZ swz) {
#pragma unroll
    for (int i = 0; i < MAXLD; ++i) {
      const int p = (lw + 4 * i) * 1024 + lane * 16, row = p / rp, inrow = p - row * rp;
      const int logi = inrow ^ (int)swz((uint32_t)inrow, row);
      goff[i] = row * rowbytes + logi - pix;
      rs[i] = p < image_bytes ? (uint32_t)row | (uint32_t)(logi / pix) << 8 : 0xffffffffu;
    }
  }
  // src: the image's pixel (iy_lo, ix0); n: this wave's loads of a tile (each has at least one lane that loads)
  template <int AUX>
  __device__ __forceinline__ void issue(const char* src, const char* zp, char* dst, int n, int lw, int iy_lo, int H, int ix0, int W) const {
#pragma unroll
    for (int i = 0; i < MAXLD; ++i)
      if (i < n) {
        const int iy = iy_lo + (int)(rs[i] & 255u), ix = ix0 - 1 + (int)(rs[i] >> 8);
        const char* p = ((uint32_t)iy < (uint32_t)H && (uint32_t)ix < (uint32_t)W) ? src + goff[i] : zp;
        if (rs[i] != 0xffffffffu) __builtin_amdgcn_global_load_lds(GLOBAL_AS(p), LDS_AS(dst + (lw + 4 * i) * 1024), 16, 0, AUX);
      }
  }
};

// The forward kernel's form for 64 channels.  A b128 operand read is served eight lanes at a time, and eight lanes
// run at full rate when their 16-byte chunks sit at eight different positions of the 128-byte pixel.  Consecutive
// lanes are consecutive output pixels, row after row of the band, so the key that permutes a pixel's chunks counts
// pixels the same way: slot pair + Wo * (image row / 2), i.e. lane number plus a constant for every tap.  (The
// in-row key alone repeats where a short output row wraps inside a group of eight lanes: 16 instead of 8 cycles
// per read at Wo = 10.)  `rowkey` = Wo * (row >> 1) of the LDS image row the byte belongs to.
template <int CIN>
__device__ __forceinline__ uint32_t fwd_swz_bits(uint32_t off, uint32_t rowkey) {
  if (CIN == 32) return tile_swz_bits<32>(off);
  if (CIN == 16) return ((off >> 8) & 1u) << 4;  // slot >> 3
  return (((off >> 8) + rowkey) & 7u) << 4;
}

// AUX: cache policy of the band loads (LOAD_NT where a band shares few rows with its neighbours); RELU = false: the sums
// pass as they are (a layer normalisation follows)
// C0 > 0 (32 input channels): the input rows are made from C0-channel images by the four waves that otherwise load them
// (conv0_rows.hip.h), one tile ahead of the compute waves, in two LDS buffers; BITS0: the mask bits of the rows are stored.
// STACK: tiles of TR rows of the batch's stacked images (common.hip.h), whole rows each.  The taps of the row above an image's
// first read zeros behind the bias table instead.
template <int CIN, int AUX, int WIDE = 0, bool RELU = true, bool COLS = false, int C0 = 0, bool BITS0 = false, bool STACK = false>
__global__ __launch_bounds__(512) void k_conv_fwd_tile(ConvTileArgs a) {
  static_assert(C0 == 0 || (CIN == 32 && RELU), "the first layer has 32 output channels");
  static_assert(!STACK || (!COLS && C0 == 0), "stacked rows are whole rows of a stored tensor");
  typedef ConvTileShape<CIN, WIDE> S;
  constexpr int NW = S::NW, WGN = S::WGN, TN = NW / 32, TM = S::TM, PIX = S::PIX, SP = S::SP;
  constexpr int KC = CIN / 16;  // MFMA k-steps per tap
  constexpr int CPP = CIN / 8;  // 16-byte chunks per pixel
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, h = lane >> 5;
  const int W = a.W, TR = a.TR, Wo = COLS ? a.TC : a.Wo, WP = COLS || C0 ? 2 * Wo + 1 : W + 2, NBUF = C0 ? 2 : a.nbuf;  // Wo: of the tile
  const int nrows = 2 * TR + 1, rowbytes = W * PIX, segs = (rowbytes + 1023) >> 10;
  const int image_bytes = C0 ? Conv0Shape1<C0>::act_bytes(Wo, TR) : nrows * WP * PIX;
  // tiles of this block: vb, vb + gridDim.x, ...
  const int vb = xcd_block((int)blockIdx.x, (int)gridDim.x);  // this block's number in the dealing of tiles
  const int nq = (a.ntiles > vb) ? (a.ntiles - 1 - vb) / (int)gridDim.x + 1 : 0;

  // zero the pad pixels of all ring images once
  if constexpr (C0 > 0) {
    for (int i = tid; i < 2 * image_bytes / 16; i += S::THREADS) reinterpret_cast<uint4*>(lds)[i] = make_uint4(0u, 0u, 0u, 0u);
  } else if constexpr (!COLS) for (int i = tid; i < NBUF * nrows * 2 * CPP; i += S::THREADS) {
    const int chunk = i % CPP, side = (i / CPP) & 1, row = i / (2 * CPP);  // row over all images
    *reinterpret_cast<uint4*>(lds + (int64_t)row * WP * PIX + (side ? (W + 1) * PIX : 0) + chunk * 16) = make_uint4(0u, 0u, 0u, 0u);
  }
  char* const zrow = lds + NBUF * image_bytes + S::STAGE_BYTES + S::BN * 4;  // STACK: three pixels of zeros
  if constexpr (STACK) {
    if (tid < 3 * CPP) *reinterpret_cast<uint4*>(zrow + tid * 16) = make_uint4(0u, 0u, 0u, 0u);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // before this wave's first barrier
  }

  if (wave >= 4) {
    // ------------------------------------------------------------------ loaders: span row r belongs to loader r % 4
    const int lw = __builtin_amdgcn_readfirstlane(wave - 4);
    if constexpr (C0 > 0) {
      // A SIMD holds one compute wave and one of these.  Where making the rows is the longer of the two (three channels, or a
      // tile's extra column), it goes first: 8400 images of 240x320 3225 -> 2790 us, 8192 stereo pairs 1438 -> 1331.  Rows of
      // one channel without tiles of columns are the shorter: 16384 images of 120x160 would go from 1176 to 1238.
      if (COLS || C0 > 1) __builtin_amdgcn_s_setprio(2);
      typedef Conv0Shape1<C0> S0;
      char* const ring = lds + 2 * image_bytes + S::STAGE_BYTES + S::BN * 4;
      const int ring_bytes = S0::image_bytes(Wo, TR), NI = a.src0.nimage, D = NI - 1, pieces = a.src0.rowbytes >> 4;
      Conv0Producer<C0, COLS, BITS0> pr;
      pr.init(a.src0, lw, lane, TR, Wo, W);
      struct Pos { int img, band, part; };
      auto pos = [&](int q) {
        const int t = vb + q * gridDim.x, tb = COLS ? (int)a.dv_np.div((uint32_t)t) : t;
        Pos p; p.part = COLS ? t - tb * a.NP : 0; p.img = (int)a.dv_nb.div((uint32_t)tb); p.band = tb - p.img * a.NB;
        return p;
      };
      int islot = 0, pslot = 0;
      typedef typename Conv0Producer<C0, COLS, BITS0>::Img Img;
      ImgAhead ahead;
      auto image = [&](int q) {
        const Pos p = pos(q);
        const int iy_lo = 4 * p.band * TR - 3, b0 = 8 * C0 * p.part * Wo;  // (Wo is even where there are several parts)
        const bf16_t* const img = ahead.ptr(a.src0.img, q, [&](int k) __attribute__((always_inline)) { return k < nq ? pos(k).img : -1; });
        const char* src = reinterpret_cast<const char*>(img) + (int64_t)iy_lo * a.src0.rowbytes + b0;
        const Img m = {src, reinterpret_cast<const char*>(a.zpage) + lane * 16, ring + islot * ring_bytes, iy_lo, a.src0.H, b0 >> 4, pieces, lw};
        islot = islot + 1 == NI ? 0 : islot + 1;
        return m;
      };
      auto produce = [&](int q) {
        const Pos p = pos(q);
        const bool edge = p.band == 0 || p.band == a.NB - 1 || (COLS && (p.part == 0 || p.part == a.NP - 1));
        const int row_lo = 2 * p.band * TR - 1, col_lo = 2 * p.part * Wo - 1;
        char* bits = BITS0 ? reinterpret_cast<char*>(a.src0.bits + ((int64_t)p.img * a.H + row_lo + 1) * a.src0.bpitch + col_lo + 1) : nullptr;
        const int st = pr.produce(ring + pslot * ring_bytes, lds + (q & 1) * image_bytes, edge, row_lo, col_lo, a.H, W, bits, [](int) {});
        pslot = pslot + 1 == NI ? 0 : pslot + 1;
        return st;
      };
      // Image q + 2 must have landed when tile q + 1 is done being made.  Behind its loads this wave has issued those of the
      // images up to q + 1 + D and the mask stores of the last D tiles it made (st[]: at least so many).
      for (int q = 0; q < D && q < nq; ++q) pr.load_all(image(q));
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      vm_wait_few((min(D, nq) - 1) * pr.nl);
      __builtin_amdgcn_s_barrier();  // the first image has landed, the buffers are zeroed
      int st0 = 0, st1 = 0, st2 = 0;
      for (int q = -1; q < nq; ++q) {
        if (q >= 0) __builtin_amdgcn_s_barrier();  // tile q is made, image q + 1 has landed
        if (q + 1 < nq) {
          if (q + 1 + D < nq) pr.load_all(image(q + 1 + D));
          __builtin_amdgcn_sched_barrier(0);
          st2 = D > 2 ? st1 : 0; st1 = st0;
          st0 = produce(q + 1);
          __builtin_amdgcn_sched_barrier(0);
          vm_wait_few(max(0, min(q + 1 + D, nq - 1) - (q + 2)) * pr.nl + st0 + st1 + st2);
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
      }
      return;
    }
    if constexpr (COLS) {
      const int ni = (((image_bytes + 1023) >> 10) - lw + 3) >> 2;  // this wave's loads per tile
      ColsLoads<S::MAXLD> ld;
      ld.init(lw, lane, image_bytes, WP * PIX, PIX, rowbytes, [&](uint32_t off, int row) { return fwd_swz_bits<CIN>(off, (uint32_t)(Wo * (row >> 1))); });
      int slot = 0;
      auto issue = [&](int q) {
        const int t = vb + q * gridDim.x, tb = (int)a.dv_np.div((uint32_t)t), part = t - tb * a.NP;
        const int img = (int)a.dv_nb.div((uint32_t)tb), band = tb - img * a.NB, iy_lo = 2 * band * TR - 1, ix0 = 2 * part * Wo;
        const char* src = reinterpret_cast<const char*>(a.in.ptr_uniform(img)) + (int64_t)iy_lo * rowbytes + ix0 * PIX;
        ld.template issue<AUX>(src, reinterpret_cast<const char*>(a.zpage) + lane * 16, lds + slot * image_bytes, ni, lw, iy_lo, a.H, ix0, W);
        slot = slot + 1 == NBUF ? 0 : slot + 1;
      };
      const int D = NBUF - 1;
      for (int q = 0; q < D && q < nq; ++q) issue(q);
      for (int q = 0; q < nq; ++q) {
        vm_wait_dyn(min(D - 1, nq - 1 - q) * ni);
        __builtin_amdgcn_s_barrier();
        if (q + D < nq) issue(q + D);
      }
      return;
    }
    const int ni = ((nrows - lw + 3) >> 2) * segs;  // this wave's loads per band
    // this lane's 16 bytes land at in-row offset PIX + sg*1024 + lane*16: it fetches what belongs there
    // (byte offset within the image row; depends on the row for 64 channels)
    auto src_off = [&](int sg, int row) {
      const uint32_t phys = PIX + sg * 1024 + lane * 16, logi = phys ^ fwd_swz_bits<CIN>(phys, (uint32_t)(Wo * (row >> 1)));
      return (sg < segs && (int)phys < (W + 1) * PIX) ? (int)logi - PIX : -1;  // -1 = none
    };
    int goff[S::MAXSEG];
#pragma unroll
    for (int sg = 0; sg < S::MAXSEG; ++sg) goff[sg] = src_off(sg, 0);
    int slot = 0;  // ring image the next issued band goes to
    auto issue = [&](int q) {
      const int t = vb + q * gridDim.x;
      const int img = STACK ? 0 : (int)a.dv_nb.div((uint32_t)t), band = t - img * a.NB;
      const int iy_lo = 2 * (STACK ? t : band) * TR - 1;
      const char* src = STACK ? reinterpret_cast<const char*>(a.in.base) : reinterpret_cast<const char*>(a.in.ptr_uniform(img)) + (int64_t)iy_lo * rowbytes;
      char* dst = lds + slot * image_bytes + PIX;  // skip the left pad
      slot = slot + 1 == NBUF ? 0 : slot + 1;
      for (int row = lw; row < nrows; row += 4) {
        const int iy = iy_lo + row;
        int mem = row;
        const bool inside = STACK ? a.stk.in_row(iy, a.H, &mem) : iy >= 0 && iy < a.H;
#pragma unroll
        for (int sg = 0; sg < S::MAXSEG; ++sg)
          if (sg < segs) {
            const int go = (CIN != 64) ? goff[sg] : src_off(sg, row);
            const char* p = inside ? src + (int64_t)mem * rowbytes + go : reinterpret_cast<const char*>(a.zpage) + lane * 16;
            if (go >= 0) __builtin_amdgcn_global_load_lds(GLOBAL_AS(p), LDS_AS(dst + row * WP * PIX + sg * 1024), 16, 0, AUX);
          }
      }
    };
    const int D = NBUF - 1;  // bands in flight
    for (int q = 0; q < D && q < nq; ++q) issue(q);
    for (int q = 0; q < nq; ++q) {
      vm_wait_dyn(min(D - 1, nq - 1 - q) * ni);  // band q has landed; the bands issued after it may still be in flight
      __builtin_amdgcn_s_barrier();
      if (q + D < nq) issue(q + D);      // into the slot the compute waves finished before this barrier
    }
    return;
  }

  // -------------------------------------------------------------------- compute waves
  const int wm = wave / WGN, wn = wave % WGN;
  char* const stage = lds + NBUF * image_bytes + wave * (32 * SP * 2);
  float* const bias_s = reinterpret_cast<float*>(lds + NBUF * image_bytes + S::STAGE_BYTES);
  const int nb0 = blockIdx.y * S::BN, n0 = nb0 + wn * NW;
  for (int i = tid; i < S::BN; i += 256) bias_s[i] = (nb0 + i < a.Cout) ? a.bias[nb0 + i] : 0.f;

  // this wave's weights, in MFMA operand layout: lane (column l32 of tile j, 8 k at h*8)
  bf16x8_t wr[9 * KC][TN];
#pragma unroll
  for (int s = 0; s < 9 * KC; ++s)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + j * 32 + l32;
      wr[s][j] = (n < a.Cout) ? *reinterpret_cast<const bf16x8_t*>(a.w + (int64_t)n * (9 * CIN) + s * 16 + h * 8)
                              : __builtin_bit_cast(bf16x8_t, make_uint4(0u, 0u, 0u, 0u));
    }

  // this lane's output pixel(s) within a band, the LDS offset of the window corner (slot 2*ox of row
  // 2*oyl) and, per tap column v, the chunk permutation of slot 2*ox + v folded with the lane's k half
  // (for 64 channels the permutation also depends on the image row pair: rows 2*oyl, 2*oyl + 1 for the taps
  // u < 2, row 2*oyl + 2 for u = 2)
  constexpr int NU = (CIN == 64) ? 2 : 1;
  uint32_t abase[TM], hx[TM][NU][3];
  uint32_t rmod = 0u;  // STACK: the pixels' rows modulo Ho, 16 bits each
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int r = (wm * TM + i) * 32 + l32;
    const bool in_band = r < TR * Wo;  // lanes beyond the band compute on pixel 0; never stored
    const int oyl = in_band ? r / Wo : 0, ox = in_band ? r - oyl * Wo : 0;
    if constexpr (STACK) rmod |= (uint32_t)a.stk.mod_ho(oyl) << (16 * i);
    abase[i] = (uint32_t)(((2 * oyl) * WP + 2 * ox) * PIX);
#pragma unroll
    for (int u2 = 0; u2 < NU; ++u2)
#pragma unroll
      for (int v = 0; v < 3; ++v)
        hx[i][u2][v] = (uint32_t)(h * 16) ^ fwd_swz_bits<CIN>((uint32_t)((2 * ox + v) * PIX), (uint32_t)(Wo * (oyl + u2)));
  }

  // COLS: row and column within the tile of the output pixels this lane writes out, row | column << 8
  constexpr int CPRO = NW / 8;  // 16-byte chunks per staged row
  uint32_t opix[TM][32 * CPRO / 64], bpix[TM];
  if constexpr (COLS) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int p0 = (wm * TM + i) * 32;
      auto rc = [&](int p) { const int r = p / Wo; return (uint32_t)r | (uint32_t)(p - r * Wo) << 8; };
      bpix[i] = rc(p0 + l32);
#pragma unroll
      for (int e = 0; e < 32 * CPRO / 64; ++e) opix[i][e] = rc(p0 + (lane + 64 * e) / CPRO);
    }
  }

  // the first tile's barrier also orders the pad fill and the bias table before their first use
  if constexpr (C0 > 0) {
    const int cpr = a.P >> 3;
    for (int i = (int)blockIdx.x * 256 + tid; i < a.n0 * cpr; i += (int)gridDim.x * 256) {
      const int b = i / cpr, j = i - b * cpr;
      const int64_t sm = a.src0.img.idx ? a.src0.img.idx[b] : b;
      reinterpret_cast<uint4*>(a.feat + (int64_t)b * a.feat_ld)[j] = reinterpret_cast<const uint4*>(a.proprio + sm * a.P)[j];
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();  // the producers' first image has landed
  }
  int slot = 0;
  for (int q = 0; q < nq; ++q) {
    const int t = vb + q * gridDim.x;
    __builtin_amdgcn_s_barrier();  // band q is in LDS
    const char* img_s = lds + slot * image_bytes;
    slot = slot + 1 == NBUF ? 0 : slot + 1;

    f32x16_t acc[TM][TN];  // starts at the bias of the lane's columns j*32 + g*8 + h*4 + 0..3
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 bv = *reinterpret_cast<const float4*>(bias_s + wn * NW + j * 32 + g * 8 + h * 4);
#pragma unroll
        for (int i = 0; i < TM; ++i) { acc[i][j][g * 4] = bv.x; acc[i][j][g * 4 + 1] = bv.y; acc[i][j][g * 4 + 2] = bv.z; acc[i][j][g * 4 + 3] = bv.w; }
      }
    // The operand reads run RD steps ahead of the MFMAs through a rotation of RD + 1 registers (step s = tap, 16-deep
    // chunk cc, pixel group i): with one compute wave per SIMD nothing else hides the LDS latency, and left to
    // itself the compiler keeps a single read in flight.  Logical chunk 2*cc + h of a slot sits at position
    // (2*cc + h) ^ f(slot, row) = (32*cc) ^ hx in bytes.
    constexpr int NS = 9 * KC * TM, RD = 3;
    const char* top[TM];  // of the window's first row
    if constexpr (STACK) {
      const int er = a.stk.edge_row(t * TR, 0);
      uint32_t rm = rmod;
      asm volatile("" : "+v"(rm));  // (not to be unpacked ahead of the loop: the wide form has no register to spare)
#pragma unroll
      for (int i = 0; i < TM; ++i) top[i] = (int)(rm >> (16 * i) & 0xffffu) == er ? zrow : img_s + abase[i];
    }
    auto operand = [&](int s) {
      const int i = s % TM, cc = (s / TM) % KC, tap = s / (TM * KC), u = tap / 3, v = tap - 3 * u;
      if (STACK && u == 0) return *reinterpret_cast<const bf16x8_t*>(top[i] + v * PIX + ((uint32_t)(cc * 32) ^ hx[i][0][v]));
      return *reinterpret_cast<const bf16x8_t*>(img_s + abase[i] + (u * WP + v) * PIX + ((uint32_t)(cc * 32) ^ hx[i][(NU == 2 && u == 2) ? 1 : 0][v]));
    };
    bf16x8_t av[RD + 1];
#pragma unroll
    for (int s = 0; s < RD; ++s) av[s] = operand(s);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      if (s + RD < NS) av[(s + RD) % (RD + 1)] = operand(s + RD);
      const int i = s % TM;
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wr[s / TM][j], av[s % (RD + 1)], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);  // keep the read of step s + RD in front of the MFMA of step s
    }
    // ---- epilogue: bf16, ReLU; lane holds pixel l32 of the wave's pixel group i, columns j*32 + g*8 + h*4 + 0..3
    // (STACK: img = 0, the band's rows are the stack's)
    const int tb = COLS ? (int)a.dv_np.div((uint32_t)t) : t, ox0 = COLS ? (t - tb * a.NP) * Wo : 0;
    const int img = STACK ? 0 : (int)a.dv_nb.div((uint32_t)tb), band = tb - img * a.NB;
    const int b = STACK ? 0 : img / a.V, vw = img - b * a.V;
    const int rows_here = min(TR, (STACK ? a.stk.rows : a.Ho) - band * TR), cols_here = min(Wo, a.Wo - ox0);
    const int plim = rows_here * Wo;  // pixels of the band that exist
    bf16_t* dst = a.out + (int64_t)b * a.out_stride_b + (int64_t)vw * a.out_stride_v + ((int64_t)band * TR * a.Wo + ox0) * a.Cout;
    // is pixel p of the tile (COLS: at row and column rc) in the image, and which pixel of the image, counted from the tile's first
    auto exists = [&](int p, uint32_t rc) { return COLS ? (int)(rc & 255u) < rows_here && (int)(rc >> 8) < cols_here : p < plim; };
    auto pix_of = [&](int p, uint32_t rc) { return COLS ? (int)(rc & 255u) * a.Wo + (int)(rc >> 8) : p; };
    const uint32_t negw = nonzero_weights(h);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int p0 = (wm * TM + i) * 32;  // the group's first pixel (the strip is reused per group: a wave's LDS
                                          // accesses are served in order)
      uint32_t pw[TN];  // this lane's 16 sign bits of the pixel's 32-column group j
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        pw[j] = 0u;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int cl = j * 32 + g * 8 + h * 4;
          uint2 o;
          o.x = RELU ? relu_pack2bf(acc[i][j][g * 4], acc[i][j][g * 4 + 1]) : pack2bf(acc[i][j][g * 4], acc[i][j][g * 4 + 1]);
          o.y = RELU ? relu_pack2bf(acc[i][j][g * 4 + 2], acc[i][j][g * 4 + 3]) : pack2bf(acc[i][j][g * 4 + 2], acc[i][j][g * 4 + 3]);
          *reinterpret_cast<uint2*>(stage + (l32 * SP + cl) * 2) = o;
          if (RELU) pw[j] |= nonzero4(o.x, o.y, negw) << (g * 8);
        }
      }
      if (RELU && a.bits) {
        // the other half of the columns sits in lane ^ 32; lanes 0..31 write the pixel's words
        const int wpp = (a.Cout + 31) >> 5, p = p0 + l32;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const uint32_t word = or_with_lane_xor32(pw[j]);
          const int wi = (n0 >> 5) + j;
          uint32_t rc = COLS ? bpix[i] : 0u;
          if (COLS) asm volatile("" : "+v"(rc));  // (its parts are not to be kept from tile to tile: the wide form has no register to spare)
          if (h == 0 && exists(p, rc) && wi < wpp)
            a.bits[((int64_t)img * a.Ho * a.Wo + (int64_t)band * TR * a.Wo + ox0 + pix_of(p, rc)) * wpp + wi] = word;
        }
      }
#pragma unroll
      for (int e = 0; e < 32 * CPRO / 64; ++e) {
        const int ch = lane + 64 * e, rl = ch / CPRO, cg = ch - rl * CPRO;
        const int p = p0 + rl, n = n0 + cg * 8;
        uint32_t rc = COLS ? opix[i][e] : 0u;
        if (COLS) asm volatile("" : "+v"(rc));
        if (exists(p, rc) && n < a.Cout) {
          const uint4 v = *reinterpret_cast<const uint4*>(stage + (rl * SP + cg * 8) * 2);
          if (STACK && !a.stk.dense) {
            const int P = t * TR * Wo + p, im = (int)a.stk.hw.div((uint32_t)P), bi = (int)a.stk.v.div((uint32_t)im);
            store_stream16(a.out + (int64_t)bi * a.out_stride_b + (int64_t)(im - bi * a.V) * a.out_stride_v + (int64_t)(P - im * (int)a.stk.hw.d) * a.Cout + n, v);
          } else
            store_stream16(dst + (int64_t)pix_of(p, rc) * a.Cout + n, v);
        }
      }
    }
  }
}

// ------------------------------------------------------------------------------------------------
// Weight gradient of the same convolution: G[n][k] = sum over pixels p of dY[p][n] * X[win(p)][k],
// k = (u*3+v)*CIN + ci, with the same organisation.  A tile is (image, band of TR output rows), or TR rows of TC columns; the
// loader waves copy the tile's input rows (LDS image as above) and its dY pixels (64 output
// channels of this block, 128 bytes per pixel, NSTEP*16 pixels with zeros beyond the tile) into a
// ring of nbuf buffers (three, or more where they fit: small bands need more of them in flight).  With C0 > 0 they load the
// first layer's images and dY alone and make the input rows, as in the forward kernel.  The contraction runs over pixels, 16
// per MFMA step; both operands are
// read through ds_read_b64_tr_b16 (lane r of a 16-lane group supplies 4 consecutive channels of
// pixel r/4, lane i receives channel i of 4 pixels), the im2col being the per-lane pixel address.
// 64 channels (18 k-tiles of 32): compute wave w owns the k-tiles w, w+4, ... of both 32-row n-tiles; waves 2 and 3
// have no fifth, and wave 3 sums the columns of dY (the bias gradient) with an all-ones operand instead.  32 channels (nine k-tiles): two whole
// k-tiles per wave; the two n-tiles of the ninth go to waves 0 and 1, those of the bias column to waves 2 and 3.
// The accumulators live in registers across all tiles of the block and leave once, as this block's fp32 partial
// [9*CIN][Cout] (partials are summed in a fixed order by the caller).
// dY pixels are 128 bytes apart; bit 6 of the offset is flipped for every second pixel pair so that
// the four pixels of one transposing read fall into different banks.
struct ConvWgradArgs {
  ImgAddr in;                 // layer input X, images [H][W][CIN], dense
  ImgAddr dy;                 // gradient of the layer output, images [Ho][Wo][Cout]
  const bf16_t* zpage;        // 1 KiB of zeros
  float* partial;             // [gridDim.x][9*CIN][Cout]
  float* bias_partial;        // [gridDim.x][Cout]
  int H, W, Ho, Wo, Cout;
  int TR, NB, ntiles, nstep;  // output rows per band, bands per image, nimg * NB, ceil(TR*Wo / 16)
  int nbuf;                   // ring buffers (3 .. MAXBUF)
  FastDiv dv_nb, dv_np;       // division by NB, NP
  int TC, NP;                 // as in ConvTileArgs
  Conv0Src src0;              // C0 > 0: where the input rows are made from
  Stack stk;                  // STACK: the batch as one tall image
};

template <int CIN>
struct ConvWgradShape {
  static constexpr int PIX = CIN * 2, KT = 9 * CIN / 32, KTW = (KT + 3) / 4;
  static constexpr int MAXSEG = 6, MAXSTEP = (CIN == 32) ? 8 : 4, MAXBUF = 6, THREADS = 512;
  static_assert(3 + 4 * (KTW - 1) >= KT, "wave 3's last accumulator pair must be free for the bias sums");
  // rounded up to 128 bytes: the dY pixels behind the image are addressed by flipping bit 6 of the whole offset (an
  // odd number of 64-byte pixel slots, i.e. an odd W at 32 channels, would leave them half a pixel off)
  // (slots: pixel slots per row, W + 2, or 2 * TC + 1 in a tile of columns)
  static constexpr int MAXLD = 13;  // COLS: 1 KiB image loads per loader wave and tile
  __host__ __device__ static int image_bytes(int slots, int TR) { return ((2 * TR + 1) * slots * PIX + 127) & ~127; }
  static int buf_bytes(int slots, int TR, int nstep) { return image_bytes(slots, TR) + nstep * 16 * 128; }
  static int lds_bytes(int slots, int TR, int nstep, int nbuf) { return nbuf * buf_bytes(slots, TR, nstep) + 4 * 64 * 4; }  // (the end: STACK's zeros)
};

// The dY pixels of a tile of columns, 64 channels each: piece j of 1 KiB belongs to loader wave j % 4.
template <int MAXDY>
struct ColsDy {
  int goff[MAXDY];     // byte offset from the tile's first pixel
  uint32_t rc[MAXDY];  // row | column << 8, ~0: zeros (such a column is in no image)
  __device__ __forceinline__ void init(int lw, int lane, int TR, int TC, int Wo, int Cout, int nb0) {
#pragma unroll
    for (int i = 0; i < MAXDY; ++i) {
      const uint32_t phys = (lw + 4 * i) * 1024 + lane * 16, logi = phys ^ (((phys >> 8) & 1u) << 6);
      const int p = (int)(logi >> 7), cb = (int)(logi & 127u), r = p / TC, cl = p - r * TC;
      goff[i] = (r * Wo + cl) * Cout * 2 + cb;
      rc[i] = (r < TR && nb0 + (cb >> 1) < Cout) ? (uint32_t)r | (uint32_t)cl << 8 : 0xffffffffu;
    }
  }
  __device__ __forceinline__ void load(const char* src, const char* zp, char* dst, int i, int lw, int oy0, int Ho, int ox0, int Wo) const {
    const bool ok = oy0 + (int)(rc[i] & 255u) < Ho && ox0 + (int)(rc[i] >> 8) < Wo;
    __builtin_amdgcn_global_load_lds(GLOBAL_AS(ok ? src + goff[i] : zp), LDS_AS(dst + (lw + 4 * i) * 1024), 16, 0, LOAD_NT);
  }
  __device__ __forceinline__ void issue(const char* src, const char* zp, char* dst, int n, int lw, int oy0, int Ho, int ox0, int Wo) const {
#pragma unroll
    for (int i = 0; i < MAXDY; ++i)
      if (i < n) load(src, zp, dst, i, lw, oy0, Ho, ox0, Wo);
  }
};

__device__ __forceinline__ bf16x8_t lds_read_tr8_2(const char* p_lo, const char* p_hi) {
  typedef short s16x4_t_ __attribute__((ext_vector_type(4)));
  struct { s16x4_t_ lo, hi; } v;
  v.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4_t_ __attribute__((address_space(3)))*)(p_lo));
  v.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4_t_ __attribute__((address_space(3)))*)(p_hi));
  return __builtin_bit_cast(bf16x8_t, v);
}

// NS > 0: the number of pixel steps per band is NS (known when the kernel is compiled), which lets the tile loop run
// without a branch and its operand reads ahead of the MFMAs; NS = 0: any number of steps up to MAXSTEP.
// COLS: tiles of columns, as in the forward kernel.  C0 > 0: the input rows are made from C0-channel images, as there; the
// ring of nbuf buffers then holds dY alone, an image travels with the dY of the tile before.
// STACK: bands of the batch's stacked images, as in the forward kernel.
template <int CIN, int NS = 0, bool COLS = false, int C0 = 0, bool STACK = false>
__global__ __launch_bounds__(512) void k_conv_wgrad_tile(ConvWgradArgs a) {
  static_assert(!STACK || (!COLS && C0 == 0), "stacked rows are whole rows of a stored tensor");
  static_assert(C0 == 0 || CIN == 32, "the first layer has 32 output channels");
  typedef ConvWgradShape<CIN> S;
  constexpr int PIX = S::PIX, KT = S::KT, KTW = S::KTW, MAXSTEP = S::MAXSTEP;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int W = a.W, TR = a.TR, Wo = COLS ? a.TC : a.Wo, WP = COLS || C0 ? 2 * Wo + 1 : W + 2, nstep = NS ? NS : a.nstep, NBUF = a.nbuf;  // Wo: of the tile
  const int nrows = 2 * TR + 1, rowbytes = W * PIX, segs = (rowbytes + 1023) >> 10;
  // (C0 > 0: two buffers of made rows, then the ring of dY buffers, then the images)
  const int image_bytes = C0 ? Conv0Shape1<C0>::act_bytes(Wo, TR) : S::image_bytes(WP, TR), dy_bytes = nstep * 16 * 128, buf_bytes = C0 ? dy_bytes : image_bytes + dy_bytes;
  const int dy_off = C0 ? 0 : image_bytes;  // of the dY pixels in a ring buffer
  char* const dyring = lds + (C0 ? 2 * image_bytes : 0);
  const int vb = xcd_block((int)blockIdx.x, (int)gridDim.x);  // this block's number in the dealing of tiles
  const int nq = (a.ntiles > vb) ? (a.ntiles - 1 - vb) / (int)gridDim.x + 1 : 0;
  const int nb0 = blockIdx.y * 64;

  // zero the pad pixels of all ring images once
  if constexpr (C0 > 0) {
    for (int i = tid; i < 2 * image_bytes / 16; i += S::THREADS) reinterpret_cast<uint4*>(lds)[i] = make_uint4(0u, 0u, 0u, 0u);
  } else if constexpr (!COLS) for (int i = tid; i < NBUF * nrows * 2 * (PIX / 16); i += S::THREADS) {
    const int chunk = i % (PIX / 16), side = (i / (PIX / 16)) & 1, row = i / (2 * (PIX / 16));
    const int b = row / nrows, rr = row - b * nrows;
    *reinterpret_cast<uint4*>(lds + b * buf_bytes + (int64_t)rr * WP * PIX + (side ? (W + 1) * PIX : 0) + chunk * 16) = make_uint4(0u, 0u, 0u, 0u);
  }
  char* const zpix = lds + NBUF * buf_bytes;  // STACK: eight bytes of zeros
  if constexpr (STACK) {
    if (tid < 4) reinterpret_cast<uint32_t*>(zpix)[tid] = 0u;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // before this wave's first barrier
  }

  if (wave >= 4) {
    // ------------------------------------------------------------------ loaders
    // loader lw copies the image rows lw, lw+4, ... and the 1 KiB dY pieces lw, lw+4, ... of a band
    const int lw = wave - 4;
    if constexpr (C0 > 0) {
      // Before the compute wave of the same SIMD, which has no vector work between its products: 16384 images of 120x160
      // 1233 -> 1180 us, 8192 stereo pairs 1645 -> 1611, 8400 images of 240x320 2882 -> 2801.
      __builtin_amdgcn_s_setprio(2);
      typedef Conv0Shape1<C0> S0;
      char* const ring = dyring + NBUF * dy_bytes;
      const int ring_bytes = S0::image_bytes(Wo, TR), D = NBUF - 1, pieces = a.src0.rowbytes >> 4;
      Conv0Producer<C0, COLS, false> pr;
      pr.init(a.src0, lw, lane, TR, Wo, W);
      ColsDy<(S::MAXSTEP * 2 + 3) / 4> dl;
      dl.init(lw, lane, TR, Wo, a.Wo, a.Cout, nb0);
      const int nd = (nstep * 2 - lw + 3) >> 2;  // this wave's dY loads per tile
      const char* const zp = reinterpret_cast<const char*>(a.zpage) + lane * 16;
      struct Pos { int img, band, part; };
      auto pos = [&](int q) {
        const int t = vb + q * gridDim.x, tb = COLS ? (int)a.dv_np.div((uint32_t)t) : t;
        Pos p; p.part = COLS ? t - tb * a.NP : 0; p.img = (int)a.dv_nb.div((uint32_t)tb); p.band = tb - p.img * a.NB;
        return p;
      };
      int islot = 0, pslot = 0, dslot = 0;
      typedef typename Conv0Producer<C0, COLS, false>::Img Img;
      ImgAhead ahead;
      auto image = [&](int q) {
        const Pos p = pos(q);
        const int iy_lo = 4 * p.band * TR - 3, b0 = 8 * C0 * p.part * Wo;
        const bf16_t* const img = ahead.ptr(a.src0.img, q, [&](int k) __attribute__((always_inline)) { return k < nq ? pos(k).img : -1; });
        const char* src = reinterpret_cast<const char*>(img) + (int64_t)iy_lo * a.src0.rowbytes + b0;
        const Img m = {src, zp, ring + islot * ring_bytes, iy_lo, a.src0.H, b0 >> 4, pieces, lw};
        islot = islot + 1 == NBUF ? 0 : islot + 1;
        return m;
      };
      struct Dy { const char* src; char* dst; int oy0, ox0; };
      auto dy_of = [&](int q) {
        const Pos p = pos(q);
        const Dy d = {reinterpret_cast<const char*>(a.dy.ptr_uniform(p.img) + ((int64_t)p.band * TR * a.Wo + p.part * Wo) * a.Cout + nb0), dyring + dslot * dy_bytes, p.band * TR, p.part * Wo};
        dslot = dslot + 1 == NBUF ? 0 : dslot + 1;
        return d;
      };
      // the loads of tile q: its dY and the image of tile q + 1
      auto issue = [&](int q) {
        const Dy d = dy_of(q);
        dl.issue(d.src, zp, d.dst, nd, lw, d.oy0, a.Ho, d.ox0, a.Wo);
        if (q + 1 < nq) pr.load_all(image(q + 1));
      };
      // Tile q from its image, the loads of tile qn (qn < nq - 1) one by one between the groups: four waves issuing all of theirs
      // at once wait hundreds of cycles for each.
      constexpr int MAXDY = (S::MAXSTEP * 2 + 3) / 4;
      auto produce = [&](int q, int qn) {
        const Pos p = pos(q);
        const bool edge = p.band == 0 || p.band == a.NB - 1 || (COLS && (p.part == 0 || p.part == a.NP - 1));
        const Dy d = dy_of(qn);
        const Img m = image(qn + 1);
        pr.produce(ring + pslot * ring_bytes, lds + (q & 1) * image_bytes, edge, 2 * p.band * TR - 1, 2 * p.part * Wo - 1, a.H, W, nullptr, [&](int g) __attribute__((always_inline)) {
          if (g < MAXDY && g < nd) dl.load(d.src, zp, d.dst, g, lw, d.oy0, a.Ho, d.ox0, a.Wo);
          if (g < pr.MAXL && g < pr.nl) pr.load(m, g);
        });
        pslot = pslot + 1 == NBUF ? 0 : pslot + 1;
      };
      auto produce_alone = [&](int q) {
        const Pos p = pos(q);
        pr.produce(ring + pslot * ring_bytes, lds + (q & 1) * image_bytes, true, 2 * p.band * TR - 1, 2 * p.part * Wo - 1, a.H, W, nullptr, [](int) {});
        pslot = pslot + 1 == NBUF ? 0 : pslot + 1;
      };
      // loads issued behind those of tile q when tiles up to q + D - 1 have been issued
      auto younger = [&](int q) { const int last = min(q + D - 1, nq - 1); return max(0, last - q) * (nd + pr.nl) - (last == nq - 1 && last > q ? pr.nl : 0); };
      // (every block has a tile)
      pr.load_all(image(0));
      for (int q = 0; q < D && q < nq; ++q) issue(q);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      vm_wait_few(younger(0) + nd + (nq > 1 ? pr.nl : 0));
      __builtin_amdgcn_s_barrier();  // the first image has landed, the buffers are zeroed
      produce_alone(0);
      const bool interleave = pr.ng > 3 ? max(nd, pr.nl) <= pr.GPW : max(nd, pr.nl) <= 3;  // as many loads of a kind as groups at most
      for (int q = 0; q < nq; ++q) {
        vm_wait_few(younger(q));       // dY of tile q and the image of tile q + 1 have landed
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();  // and tile q is made
        if (interleave && q + D + 1 < nq) produce(q + 1, q + D);
        else {
          if (q + D < nq) issue(q + D);
          if (q + 1 < nq) produce_alone(q + 1);
        }
      }
      __builtin_amdgcn_s_barrier();  // pairs with the compute waves' barrier before the bias reduction
      return;
    }
    if constexpr (COLS) {
      const int xbytes = nrows * WP * PIX;
      const int nx = (((xbytes + 1023) >> 10) - lw + 3) >> 2, ni = nx + ((nstep * 2 - lw + 3) >> 2);  // this wave's loads per tile
      ColsLoads<S::MAXLD> ld;
      ld.init(lw, lane, xbytes, WP * PIX, PIX, rowbytes, [&](uint32_t off, int) { return tile_swz_bits<CIN>(off); });
      ColsDy<(S::MAXSTEP * 2 + 3) / 4> dl;
      dl.init(lw, lane, TR, Wo, a.Wo, a.Cout, nb0);
      int slot = 0;
      auto issue = [&](int q) {
        const int t = vb + q * gridDim.x, tb = (int)a.dv_np.div((uint32_t)t), part = t - tb * a.NP;
        const int img = (int)a.dv_nb.div((uint32_t)tb), band = tb - img * a.NB, iy_lo = 2 * band * TR - 1, ox0 = part * Wo;
        const char* zp = reinterpret_cast<const char*>(a.zpage) + lane * 16;
        char* buf = lds + slot * buf_bytes;
        slot = slot + 1 == NBUF ? 0 : slot + 1;
        ld.template issue<LOAD_NT>(reinterpret_cast<const char*>(a.in.ptr_uniform(img)) + (int64_t)iy_lo * rowbytes + 2 * ox0 * PIX, zp, buf, nx, lw, iy_lo, a.H, 2 * ox0, W);
        const char* dsrc = reinterpret_cast<const char*>(a.dy.ptr_uniform(img) + ((int64_t)band * TR * a.Wo + ox0) * a.Cout + nb0);
        dl.issue(dsrc, zp, buf + image_bytes, ni - nx, lw, band * TR, a.Ho, ox0, a.Wo);
      };
      const int D = NBUF - 1;
      for (int q = 0; q < D && q < nq; ++q) issue(q);
      for (int q = 0; q < nq; ++q) {
        vm_wait_dyn(min(D - 1, nq - 1 - q) * ni);
        __builtin_amdgcn_s_barrier();
        if (q + D < nq) issue(q + D);
      }
      __builtin_amdgcn_s_barrier();  // pairs with the compute waves' barrier before the bias reduction
      return;
    }
    const int ni = ((nrows - lw + 3) >> 2) * segs + ((nstep * 2 - lw + 3) >> 2);  // this wave's loads per band
    int xgoff[S::MAXSEG];
#pragma unroll
    for (int sg = 0; sg < S::MAXSEG; ++sg) {
      const uint32_t phys = PIX + sg * 1024 + lane * 16, logi = phys ^ tile_swz_bits<CIN>(phys);
      xgoff[sg] = (sg < segs && (int)phys < (W + 1) * PIX) ? (int)logi - PIX : -1;
    }
    int slot = 0;  // ring buffer the next issued band goes to
    auto issue = [&](int q) {
      const int t = vb + q * gridDim.x;
      const int img = STACK ? 0 : (int)a.dv_nb.div((uint32_t)t), band = STACK ? t : t - img * a.NB;
      const int iy_lo = 2 * band * TR - 1;
      const char* xsrc = STACK ? reinterpret_cast<const char*>(a.in.base) : reinterpret_cast<const char*>(a.in.ptr_uniform(img)) + (int64_t)iy_lo * rowbytes;
      const int plim = min(TR, (STACK ? a.stk.rows : a.Ho) - band * TR) * Wo;  // pixels of the band that exist
      const bf16_t* dsrc = (STACK ? a.dy.base : a.dy.ptr_uniform(img)) + (int64_t)band * TR * Wo * a.Cout + nb0;
      char* buf = lds + slot * buf_bytes;
      slot = slot + 1 == NBUF ? 0 : slot + 1;
      const char* zp = reinterpret_cast<const char*>(a.zpage) + lane * 16;
      for (int row = lw; row < nrows; row += 4) {
        const int iy = iy_lo + row;
        int mem = row;
        const bool inside = STACK ? a.stk.in_row(iy, a.H, &mem) : iy >= 0 && iy < a.H;
#pragma unroll
        for (int sg = 0; sg < S::MAXSEG; ++sg)
          if (sg < segs) {
            const char* p = inside ? xsrc + (int64_t)mem * rowbytes + xgoff[sg] : zp;
            if (xgoff[sg] >= 0) __builtin_amdgcn_global_load_lds(GLOBAL_AS(p), LDS_AS(buf + row * WP * PIX + PIX + sg * 1024), 16, 0, LOAD_NT);
          }
      }
      for (int j = lw; j < nstep * 2; j += 4) {  // 1 KiB = 8 pixels of 128 bytes
        const uint32_t phys = j * 1024 + lane * 16, logi = phys ^ (((phys >> 8) & 1u) << 6);
        const int p_ = (int)(logi >> 7), cb = (int)(logi & 127u);
        const bool ok = p_ < plim && nb0 + (cb >> 1) < a.Cout;
        const char* p = ok ? reinterpret_cast<const char*>(dsrc + (int64_t)p_ * a.Cout) + cb : zp;
        if (STACK && !a.stk.dense) {
          const int P = ok ? band * TR * Wo + p_ : 0, im = (int)a.stk.hw.div((uint32_t)P), bi = (int)a.stk.v.div((uint32_t)im);
          const bf16_t* const d = a.dy.base + (int64_t)bi * a.dy.stride_b + (int64_t)(im - bi * a.dy.V) * a.dy.stride_v + (int64_t)(P - im * (int)a.stk.hw.d) * a.Cout + nb0;
          p = ok ? reinterpret_cast<const char*>(d) + cb : zp;
        }
        __builtin_amdgcn_global_load_lds(GLOBAL_AS(p), LDS_AS(buf + image_bytes + j * 1024), 16, 0, LOAD_NT);
      }
    };
    const int D = NBUF - 1;  // bands in flight
    for (int q = 0; q < D && q < nq; ++q) issue(q);
    for (int q = 0; q < nq; ++q) {
      vm_wait_dyn(min(D - 1, nq - 1 - q) * ni);  // band q has landed; the bands issued after it may still be in flight
      __builtin_amdgcn_s_barrier();
      if (q + D < nq) issue(q + D);
    }
    __builtin_amdgcn_s_barrier();  // pairs with the compute waves' barrier before the bias reduction
    return;
  }

  // -------------------------------------------------------------------- compute waves
  const int g = lane >> 4, r16 = lane & 15;
  const int scolb = (16 * (g & 1) + 4 * (r16 & 3)) * 2;  // byte offset of this lane's 4 source channels in a 32-channel tile
  // 32 channels: nine k-tiles and the bias column, two halves of 32 gradient channels each, are five MFMAs a step for each of
  // the four waves (two whole k-tiles; the ninth's halves on waves 0 and 1, the bias column's on waves 2 and 3) instead of six,
  // a sixth of which computed nothing.  Odd waves take the halves the other way round, so that the single one is always
  // the first.  16384 images of 120x160: 1291 -> 1249 us, 8192 stereo pairs 1652 -> 1594, 8400 images of 240x320 2968 -> 2857.
  // (64 channels: 38 such products, ten per wave either way.)
  constexpr bool HALF = CIN == 32;
  const uint32_t nsw = HALF ? (uint32_t)(wave & 1) : 0u;
  const bool bias_wave = HALF ? wave >= 2 : wave == 3;
  // per step and half (pixels +0..3 / +4..7 of the lane's group): source addresses within a ring buffer
  uint32_t xb[MAXSTEP][2][2];  // image: pixel (2*oyl, 2*ox) with the chunk permutation of tap columns v < 2 / v = 2
  uint32_t db[MAXSTEP][2];     // dY: pixel p, n-tile nsw
  uint32_t rmod[MAXSTEP / 2];  // STACK: the pixels' rows modulo Ho, eight bits each
#pragma unroll
  for (int i = 0; i < MAXSTEP / 2; ++i) rmod[i] = 0u;
#pragma unroll
  for (int s = 0; s < MAXSTEP; ++s)
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      int p = s * 16 + 8 * (g >> 1) + (r16 >> 2) + 4 * hf;
      const uint32_t dl = (uint32_t)(p * 128 + scolb);
      db[s][hf] = (uint32_t)dy_off + (dl ^ (((dl >> 8) & 1u) << 6) ^ nsw * 64u);
      if (p >= TR * Wo) p = 0;  // its dY is zero; any finite pixel will do
      const int oyl = p / Wo, ox = p - oyl * Wo;
      if constexpr (STACK) rmod[s / 2] |= (uint32_t)a.stk.mod_ho(oyl) << (16 * (s & 1) + 8 * hf);
      const uint32_t inrow = (uint32_t)(2 * ox * PIX + scolb), rowb = (uint32_t)(2 * oyl * WP * PIX);
      xb[s][hf][0] = rowb + (inrow ^ tile_swz_bits<CIN>(inrow));
      xb[s][hf][1] = rowb + (inrow ^ tile_swz_bits<CIN>(inrow + 2 * PIX));
    }

  f32x16_t acc[KTW][2];  // bias waves have no k-tile for t = KTW-1: that pair (HALF: its first) holds the bias sums
#pragma unroll
  for (int t = 0; t < KTW; ++t)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[t][i][e] = 0.f;
  const bf16x8_t ones = __builtin_bit_cast(bf16x8_t, make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u));
  // byte offset of k-tile kt within the window: tap (u, v) and, for 64 channels, the pixel half
  uint32_t tapc[KTW]; bool tapv2[KTW], taphi[KTW];
  int tapu0[KTW];  // STACK: 0 where the tap reads the window's first row, else a number that no row has
#pragma unroll
  for (int t = 0; t < KTW; ++t) {
    // (a wave without a k-tile for t = KTW-1 reads its first one again where the loop has no branch: the product
    // lands in an accumulator that is never stored, or is replaced by the bias operand)
    const int kt = HALF && t == KTW - 1 ? KT - 1 : (wave + 4 * t < KT) ? wave + 4 * t : wave, tap = kt / (CIN / 32), u = tap / 3, v = tap - 3 * u;
    tapc[t] = (uint32_t)((u * WP + v) * PIX); tapv2[t] = v == 2; taphi[t] = (CIN == 64) && (kt & 1);
    tapu0[t] = u == 0 ? 0 : -(1 << 20);
  }

  if constexpr (C0 > 0) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();  // the producers' first image has landed
  }
  int slot = 0;
  for (int q = 0; q < nq; ++q) {
    __builtin_amdgcn_s_barrier();  // band q is in LDS (the first one also orders the pad fill)
    const char* dbuf = dyring + slot * buf_bytes;
    const char* buf = C0 ? lds + (q & 1) * image_bytes : dbuf;
    slot = slot + 1 == NBUF ? 0 : slot + 1;
    const int er = STACK ? a.stk.edge_row((vb + q * (int)gridDim.x) * TR, 0) : 0;  // a pixel of that row (modulo Ho) has no row above
    uint32_t rm[MAXSTEP / 2];
#pragma unroll
    for (int i = 0; i < MAXSTEP / 2; ++i) {
      rm[i] = rmod[i];
      if (STACK) asm volatile("" : "+v"(rm[i]));  // (not to be unpacked ahead of the loop: there is no register to spare)
    }
    // does half hf of step s lie in row e?
    auto in_row = [&](int s, int hf, int e) __attribute__((always_inline)) { return (int)(rm[s / 2] >> (16 * (s & 1) + 8 * hf) & 255u) == e; };
    if constexpr (NS > 0) {
      // The operand reads run ahead of the MFMAs (the window operand RD k-tiles, the dY operand a whole pixel
      // step): with one compute wave per SIMD nothing else hides the LDS latency, and left to itself the compiler
      // waits for each read right where it is used.  No branch inside: every wave runs KTW k-tiles per step.
      constexpr int NU = NS * KTW, RD = 2;
      bf16x8_t aq[2][2], bq[RD + 1];
      const uint32_t bias_sel = bias_wave ? 0xffffffffu : 0u;  // a bias wave's last k-tile is the bias column
      auto read_a = [&](int s_) __attribute__((always_inline)) {
        aq[s_ & 1][0] = lds_read_tr8_2(dbuf + db[s_][0], dbuf + db[s_][1]);
        aq[s_ & 1][1] = lds_read_tr8_2(dbuf + (db[s_][0] ^ 64u), dbuf + (db[s_][1] ^ 64u));
      };
      auto read_b = [&](int u) __attribute__((always_inline)) {
        const int s_ = u / KTW, t_ = u % KTW;
        uint32_t o0 = tapv2[t_] ? xb[s_][0][1] : xb[s_][0][0], o1 = tapv2[t_] ? xb[s_][1][1] : xb[s_][1][0];
        const uint32_t hi = taphi[t_] ? 64u : 0u;
        o0 ^= hi; o1 ^= hi;
        const char *p0 = buf + o0 + tapc[t_], *p1 = buf + o1 + tapc[t_];
        if (STACK) { const int e = er + tapu0[t_]; p0 = in_row(s_, 0, e) ? zpix : p0; p1 = in_row(s_, 1, e) ? zpix : p1; }
        bq[u % (RD + 1)] = lds_read_tr8_2(p0, p1);
      };
      read_a(0);
#pragma unroll
      for (int u = 0; u < RD && u < NU; ++u) read_b(u);
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const int s_ = u / KTW, t = u % KTW;
        if (t == 0 && s_ + 1 < NS) read_a(s_ + 1);
        if (u + RD < NU) read_b(u + RD);
        bf16x8_t bop = bq[u % (RD + 1)];
        if (t == KTW - 1) {
          const uint4 bu = __builtin_bit_cast(uint4, bop), on = __builtin_bit_cast(uint4, ones);
          bop = __builtin_bit_cast(bf16x8_t, make_uint4((bu.x & ~bias_sel) | (on.x & bias_sel), (bu.y & ~bias_sel) | (on.y & bias_sel),
                                                         (bu.z & ~bias_sel) | (on.z & bias_sel), (bu.w & ~bias_sel) | (on.w & bias_sel)));
        }
        acc[t][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aq[s_ & 1][0], bop, acc[t][0], 0, 0, 0);
        if (!HALF || t < KTW - 1) acc[t][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aq[s_ & 1][1], bop, acc[t][1], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);  // keep the reads in front of the MFMAs they run ahead of
      }
    } else {
#pragma unroll
    for (int s = 0; s < MAXSTEP; ++s) {
      if (s < nstep) {
        const bf16x8_t a0 = lds_read_tr8_2(dbuf + db[s][0], dbuf + db[s][1]);
        const bf16x8_t a1 = lds_read_tr8_2(dbuf + (db[s][0] ^ 64u), dbuf + (db[s][1] ^ 64u));
#pragma unroll
        for (int t = 0; t < KTW; ++t) {
          if (HALF && t == KTW - 1 ? !bias_wave : wave + 4 * t < KT) {
            uint32_t o0 = tapv2[t] ? xb[s][0][1] : xb[s][0][0], o1 = tapv2[t] ? xb[s][1][1] : xb[s][1][0];
            if (taphi[t]) { o0 ^= 64u; o1 ^= 64u; }
            const char *p0 = buf + o0 + tapc[t], *p1 = buf + o1 + tapc[t];
            if (STACK) { const int e = er + tapu0[t]; p0 = in_row(s, 0, e) ? zpix : p0; p1 = in_row(s, 1, e) ? zpix : p1; }
            const bf16x8_t b = lds_read_tr8_2(p0, p1);
            acc[t][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, b, acc[t][0], 0, 0, 0);
            if (!HALF || t < KTW - 1) acc[t][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, b, acc[t][1], 0, 0, 0);
          }
        }
        if (bias_wave && a.bias_partial) {
          acc[KTW - 1][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, ones, acc[KTW - 1][0], 0, 0, 0);
          if (!HALF) acc[KTW - 1][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, ones, acc[KTW - 1][1], 0, 0, 0);
        }
      }
    }
    }
  }
  // ---- this block's partial sums: acc[t][i][e] = G[n][k], k = (wave+4t)*32 + lane%32 (HALF, the last t: of k-tile KT-1),
  // n = nb0 + (i^nsw)*32 + (e/4)*8 + (lane/32)*4 + e%4.
  // The partial is stored k-major ([9*CIN][Cout]) so that a lane's four consecutive n leave as one 16-byte store
  // (a quarter of the store instructions; the reduction kernel transposes back).
  const int K = 9 * CIN;
  float* P = a.partial + (int64_t)blockIdx.x * a.Cout * K;
#pragma unroll
  for (int t = 0; t < KTW; ++t) {
    const bool single = HALF && t == KTW - 1;
    const int kt = single ? (bias_wave ? KT : KT - 1) : wave + 4 * t, k = kt * 32 + (lane & 31);
    if (kt < KT) {
#pragma unroll
      for (int i = 0; i < (single ? 1 : 2); ++i)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
          const int n = nb0 + (i ^ (int)nsw) * 32 + g4 * 8 + (lane >> 5) * 4;
          if (n < a.Cout)  // Cout is a multiple of 8
            *reinterpret_cast<float4*>(P + (int64_t)k * a.Cout + n) = make_float4(acc[t][i][g4 * 4], acc[t][i][g4 * 4 + 1], acc[t][i][g4 * 4 + 2], acc[t][i][g4 * 4 + 3]);
        }
    }
  }
  __builtin_amdgcn_s_barrier();
  if (bias_wave && a.bias_partial && (lane & 31) == 0) {
    // every column of the pair holds the same sums; lanes 0 and 32 cover the 64 rows between them
#pragma unroll
    for (int i = 0; i < (HALF ? 1 : 2); ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int n = nb0 + (i ^ (int)nsw) * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
        if (n < a.Cout) a.bias_partial[(int64_t)blockIdx.x * a.Cout + n] = acc[KTW - 1][i][e];
      }
  }
}
